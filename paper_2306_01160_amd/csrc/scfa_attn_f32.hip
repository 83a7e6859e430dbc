// fp32 forward attention over the work list, on the fp32 matrix instructions (v_mfma_f32_32x32x2_f32: products and
// sums in full fp32), with the running maximum / sum recurrence of paper App. B.1 and an un-normalised accumulator
// that is divided by the sum once at the end.
//
// A workgroup owns one work item of 64 query rows: two wavefronts of 32 rows (a row per lane, as in the bf16 kernel:
// S^T = K Q^T leaves a row's scores in its lane, and S^T's accumulator layout is the B operand of O^T += V^T P^T), times
// KS key splits: split ks walks the key tiles ks, ks + KS, ... with a running maximum, sum and accumulator of its own, and
// the splits are put together through LDS at the end.  The matrix pipe bounds a tile (32 queries x 32 keys x d = 64: 64
// instructions of 64 cycles), so a short item costs its serial chain of tiles; the splits divide the chain.  Latency is
// hidden by other workgroups, four per CU at d = 64: 128 registers and 33 KB of LDS, single-buffered.  (Four splits with
// the next step's rows in registers: 170 registers, one workgroup of eight wavefronts per CU, 25 us slower.)
// Measured, hash-sparse forward on 32 segments of 2048 rows in 8 buckets, d = 64: 289 us with one thread per query row
// (vector units, one key at a time), 55 us now; one segment of 256 rows in 4 buckets: 65 and 10 us.
//
// Rows come either permuted or straight from the tensors in original order, through the positions in the sort keys
// (INDIRECT): fp32 needs no conversion, so permuted copies would only cost their traffic.
//
// The products with V take every key of a tile, masked ones with probability 0, and 0 * inf is no number: a value of a masked
// key that is not finite would reach the row.  Such items show (a result is not finite) and are done again: V without those
// values, which are then added to the rows that attend their keys.
//
// A key that is masked for a row scores -inf there; a row that never takes a key keeps m = -inf and l = 0 and writes a
// zero vector and LSE = -inf, the paper's treatment of stranded queries (Sec. 3.1 "Edge cases").
#include "scfa_common.hpp"
#include "scfa_mma.hpp"

#include <math.h>

namespace scfa {

constexpr int F32_QW = F32_TILE_M / 32;   // wavefronts side by side over the query rows of an item

__device__ __forceinline__ f32x16 mfma_f32(float a, float b, f32x16 c)
{
    return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}

template <int D, int KS>
struct F32Tiles {
    static constexpr int THREADS = F32_QW * KS * 64;
    static constexpr int ROWS = F32_TILE_N * KS;                  // keys per step of the workgroup
    static constexpr int CH = D / 4;                              // 16-byte chunks per row
    static constexpr int RPT = ROWS * CH / THREADS;               // chunks (of K, and of V) per thread and step
    static constexpr int RPR = THREADS / CH;                      // rows one round of the workgroup covers
    static constexpr int V_OFF = ROWS * D;                        // float offsets in LDS
    static constexpr int KEY_OFF = 2 * ROWS * D;
    static constexpr int SMEM = (2 * ROWS * D + ROWS + 4) * 4;    // K, V, keys, a flag per query wavefront
    static constexpr int MERGE = (D / 2 + 2) * 64;                // floats a wavefront hands over when splits are put together
    static_assert(MERGE * F32_QW * (KS / 2) * 4 <= SMEM, "the splits are put together in the tiles' LDS");
};

// on the bits, and hidden from the compiler, which may take it that there is no NaN (-fno-honor-nans)
__device__ __forceinline__ bool is_finite(float x)
{
    uint32_t u = __float_as_uint(x);
    touch(u);
    return (u & 0x7f800000u) != 0x7f800000u;
}
__device__ __forceinline__ float finite_or_zero(float x) { return is_finite(x) ? x : 0.f; }

// K is read 16 rows x one chunk at a time, V as 32 consecutive floats of rows r (lanes 0-31) and r + 4 (lanes 32-63):
// each must land on distinct banks (a row of 64 floats is one line of the 64 banks)
__device__ __forceinline__ int f32_k_chunk(int row, int c) { return c ^ (row & 15); }
__device__ __forceinline__ int f32_v_chunk(int row, int c) { return c ^ (((row >> 2) & 1) << 3); }

template <int D, int KS, bool INDIRECT>
__global__ __launch_bounds__(F32_QW * KS * 64) __attribute__((amdgpu_waves_per_eu(D == 64 ? 4 : 2))) void attn_fwd_f32_kernel(
    const float* __restrict__ q, const float* __restrict__ k, const float* __restrict__ v,
    const uint32_t* __restrict__ q_key, const uint32_t* __restrict__ k_key,
    const int32_t* __restrict__ work, int n_work, int first, int S, int T, float tau, int strict, float* __restrict__ o,
    float* __restrict__ lse, const int32_t* __restrict__ n_keep_q)
{
    using L = F32Tiles<D, KS>;
    extern __shared__ __attribute__((aligned(16))) float f32_smem[];
    float* Ks = f32_smem;
    float* Vs = f32_smem + L::V_OFF;
    uint32_t* keys_s = reinterpret_cast<uint32_t*>(f32_smem + L::KEY_OFF);

    const int s = blockIdx.x % S;
    const int w = first + blockIdx.x / S;
    const size_t seg = (size_t)s * T;
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, l32 = lane & 31, h = lane >> 5;
    if (n_keep_q) {   // QK-dropping: a share of the segment's dropped rows (zeros, LSE = -inf)
        const int sub = tid / L::CH, c = tid % L::CH;
        for (long long r = (long long)n_keep_q[s] + (long long)w * L::RPR + sub; r < T; r += (long long)n_work * L::RPR) {
            const size_t pos = seg + (q_key[seg + r] & KEY_POS_MASK);
            reinterpret_cast<float4*>(o + pos * D)[c] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (c == 0) lse[pos] = -INFINITY;
        }
    }
    const int32_t* it = work + ((size_t)s * n_work + w) * WORK_STRIDE;
    const int q_begin = it[W_QBEGIN], q_count = it[W_QCOUNT];
    const int k_begin = it[W_KBEGIN], k_count = it[W_KCOUNT];
    if (q_count <= 0) return;

    const int qw = wave % F32_QW, ks = wave / F32_QW;
    const int n_steps = (k_count + L::ROWS - 1) / L::ROWS;
    const uint32_t* kkeys = k_key + seg + k_begin;

    // one segment of K and of V (its bytes stay below 2^31)
    const auto k_rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(k + seg * D), 0, T * D * 4, 0x00020000);
    const auto v_rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(v + seg * D), 0, T * D * 4, 0x00020000);
    uint32_t nkey[L::RPT];            // sort keys of the rows of the next step
    auto load_keys = [&](int step, int trow) {
#pragma unroll
        for (int i = 0; i < L::RPT; ++i) {
            const int r = step * L::ROWS + i * L::RPR + trow;
            nkey[i] = r < k_count ? kkeys[r] : KEY_PAST_END;
        }
    };
    load_keys(0, tid / L::CH);

    const int qrow = qw * 32 + l32;
    const bool valid = qrow < q_count;
    const int qr = min(qrow, q_count - 1);            // rows past the end repeat the last one; never written
    const uint32_t qkey = q_key[seg + q_begin + qr];
    const int qpos = (int)(qkey & KEY_POS_MASK);
    // a key is taken iff (its sort key - qlo) <= qspan: same bucket, position <= the query's (< if strict)
    const bool some = valid && qpos - strict >= 0;
    const uint32_t qlo = some ? (qkey & ~KEY_POS_MASK) : KEY_NEVER;
    const uint32_t qspan = some ? (uint32_t)(qpos - strict) : 0u;
    // the sort keys any query of this wavefront may take lie in [qlo_wave, qhi_wave]
    uint32_t qlo_wave = some ? qlo : 0xffffffffu, qhi_wave = some ? qlo + qspan : 0u;
#pragma unroll
    for (int off = 16; off > 0; off >>= 1) {
        qlo_wave = min(qlo_wave, (uint32_t)__shfl_xor((int)qlo_wave, off));
        qhi_wave = max(qhi_wave, (uint32_t)__shfl_xor((int)qhi_wave, off));
    }
    qlo_wave = __builtin_amdgcn_readfirstlane(qlo_wave);
    qhi_wave = __builtin_amdgcn_readfirstlane(qhi_wave);

    f32x16 acc[D / 32];
    const float cexp = tau * LOG2E;    // probabilities are 2^(cexp (s - m)) of the raw scores <q, k>
    float m, l;                        // m: raw, so that the logsumexp has the bits of tau m; l: this lane's half of the sum
    // Once, and again without the values that are not finite where a result is not (0 * inf in the products of masked keys, see
    // above): their rows then get them added.  Unrolled: a test of which it is, between the requests of a step's rows and their way
    // into LDS, cost 3-7 % at d = 128.
#pragma unroll
    for (int again = 0; again < 2; ++again) {
#pragma unroll
        for (int db = 0; db < D / 32; ++db) acc[db] = zero16();
        m = -INFINITY;
        l = 0.f;
        // what follows from the thread's place is derived in either pass: kept from the first one to the second it costs spills
        int place = tid;
        touch(place);
        const int l32 = place & 31, h = (place >> 5) & 1;
        // rows of this thread in a step: round i covers rows i * RPR + tid / CH
        const int trow = place / L::CH, tch = place % L::CH;
        // contraction slot of lane half h in step e: element h D/2 + e of the row
        float qf[D / 2];
        {
            int row = INDIRECT ? qpos : q_begin + qr;
            touch(row);
            const float4* src = reinterpret_cast<const float4*>(q + (seg + row) * D + h * (D / 2));
#pragma unroll
            for (int c = 0; c < D / 8; ++c) {
                const float4 t = src[c];
                qf[4 * c] = t.x; qf[4 * c + 1] = t.y; qf[4 * c + 2] = t.z; qf[4 * c + 3] = t.w;
            }
        }
        for (int step = 0; step < n_steps; ++step) {
            float4 kreg[L::RPT], vreg[L::RPT];
#pragma unroll
            for (int i = 0; i < L::RPT; ++i) {
                const int r = step * L::ROWS + i * L::RPR + trow;
                const int row = INDIRECT ? (int)(nkey[i] & KEY_POS_MASK) : k_begin + r;
                const int off = r < k_count ? (row * L::CH + tch) * 16 : -1;       // out of the descriptor's range: zeros
                kreg[i] = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(k_rsrc, off, 0, 0));
                vreg[i] = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(v_rsrc, off, 0, 0));
            }
            if (again) {
#pragma unroll
                for (int i = 0; i < L::RPT; ++i)
                    vreg[i] = make_float4(finite_or_zero(vreg[i].x), finite_or_zero(vreg[i].y), finite_or_zero(vreg[i].z), finite_or_zero(vreg[i].w));
            }
            __syncthreads();               // everyone has left the previous step's tiles
#pragma unroll
            for (int i = 0; i < L::RPT; ++i) {
                const int r = i * L::RPR + trow;
                reinterpret_cast<float4*>(Ks + r * D)[f32_k_chunk(r, tch)] = kreg[i];
                reinterpret_cast<float4*>(Vs + r * D)[f32_v_chunk(r, tch)] = vreg[i];
                if (tch == 0) keys_s[r] = nkey[i];
            }
            load_keys(step + 1, trow);           // past the end: no loads
            __syncthreads();

            const int base = ks * F32_TILE_N;      // this split's tile
            if (step * L::ROWS + base >= k_count) continue;
            const int last = min(F32_TILE_N, k_count - step * L::ROWS - base) - 1;
            if ((uint32_t)__builtin_amdgcn_readfirstlane(keys_s[base]) > qhi_wave ||
                (uint32_t)__builtin_amdgcn_readfirstlane(keys_s[base + last]) < qlo_wave)
                continue;                          // nothing for the rows of this wavefront (keys ascend)

            f32x16 sacc = zero16();
#pragma unroll
            for (int c = 0; c < D / 8; ++c) {
                const float4 a = reinterpret_cast<const float4*>(Ks + (base + l32) * D)[f32_k_chunk(l32, h * (D / 8) + c)];
                sacc = mfma_f32(a.x, qf[4 * c], sacc);
                sacc = mfma_f32(a.y, qf[4 * c + 1], sacc);
                sacc = mfma_f32(a.z, qf[4 * c + 2], sacc);
                sacc = mfma_f32(a.w, qf[4 * c + 3], sacc);
            }
            float mx = -INFINITY;
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const uint4 kp = *reinterpret_cast<const uint4*>(&keys_s[base + 8 * g + 4 * h]);
                const uint32_t kv[4] = {kp.x, kp.y, kp.z, kp.w};
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    sacc[4 * g + e] = kv[e] - qlo > qspan ? -INFINITY : sacc[4 * g + e];          // bucket and causal test
                    mx = fmaxf(mx, sacc[4 * g + e]);
                }
            }
            const float m_new = fmaxf(m, half_max(mx));
            const float m_use = m_new == -INFINITY ? 0.f : m_new;
            const float alpha = fast_exp2((m - m_use) * cexp);   // m = -inf until the first taken key -> 0
            m = m_new;
            float sum = 0.f;
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                sacc[i] = fast_exp2((sacc[i] - m_use) * cexp);
                sum += sacc[i];
            }
            l = l * alpha + sum;
#pragma unroll
            for (int db = 0; db < D / 32; ++db)
#pragma unroll
                for (int i = 0; i < 16; ++i) acc[db][i] *= alpha;
            // register i of the lane is key 8 (i / 4) + 4 h + i % 4: the contraction slot of its half
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const int r = 8 * (i >> 2) + 4 * h + (i & 3);
#pragma unroll
                for (int db = 0; db < D / 32; ++db) {
                    const int c = db * 32 + l32;
                    acc[db] = mfma_f32(Vs[(base + r) * D + f32_v_chunk(r, c >> 2) * 4 + (c & 3)], sacc[i], acc[db]);
                }
            }
        }

        // put the key splits together: the upper half of them hands over, the lower half adds
#pragma unroll
        for (int half = KS / 2; half > 0; half /= 2) {
            float* mine = f32_smem + ((ks % half) * F32_QW + qw) * L::MERGE + lane;
            __syncthreads();
            if (ks >= half && ks < 2 * half) {
                mine[0] = m;
                mine[64] = l;
#pragma unroll
                for (int db = 0; db < D / 32; ++db)
#pragma unroll
                    for (int i = 0; i < 16; ++i) mine[(2 + db * 16 + i) * 64] = acc[db][i];
            }
            __syncthreads();
            if (ks < half) {
                const float m2 = mine[0], l2 = mine[64];
                const float m_new = fmaxf(m, m2);
                const float m_use = m_new == -INFINITY ? 0.f : m_new;
                const float a1 = fast_exp2((m - m_use) * cexp), a2 = fast_exp2((m2 - m_use) * cexp);
                m = m_new;
                l = l * a1 + l2 * a2;
#pragma unroll
                for (int db = 0; db < D / 32; ++db)
#pragma unroll
                    for (int i = 0; i < 16; ++i) acc[db][i] = acc[db][i] * a1 + mine[(2 + db * 16 + i) * 64] * a2;
            }
        }
        if (again) {
            if (ks == 0) {
                for (int r = 0; r < k_count; ++r) {
                    const uint32_t key = kkeys[r];
                    if (key - qlo > qspan) continue;
                    const float* row = v + (seg + (INDIRECT ? (size_t)(key & KEY_POS_MASK) : (size_t)(k_begin + r))) * D + 4 * h;
#pragma unroll
                    for (int db = 0; db < D / 32; ++db)
#pragma unroll
                        for (int g = 0; g < 4; ++g) {
                            const float4 x = *reinterpret_cast<const float4*>(row + db * 32 + 8 * g);
                            const float e[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
                            for (int i = 0; i < 4; ++i)
                                if (!is_finite(e[i])) acc[db][4 * g + i] += e[i];
                        }
                }
            }
            break;
        }
        uint32_t largest = 0;                      // of the magnitudes' bits
#pragma unroll
        for (int db = 0; db < D / 32; ++db)
#pragma unroll
            for (int i = 0; i < 16; ++i) largest = max(largest, __float_as_uint(acc[db][i]) & 0x7fffffffu);
        const bool bad = __ballot(largest >= 0x7f800000u) != 0;
        uint32_t* const bad_s = keys_s + L::ROWS;
        if (ks == 0 && lane == 0) bad_s[qw] = bad;
        __syncthreads();
        uint32_t any = 0;
#pragma unroll
        for (int i = 0; i < F32_QW; ++i) any |= bad_s[i];
        if (!__builtin_amdgcn_readfirstlane(any)) break;
        load_keys(0, trow);
    }
    if (ks != 0 || !valid) return;
    const float ltot = half_sum(l);
    const float inv = ltot > 0.f ? 1.f / ltot : 0.f;
    float* dst = o + (seg + qpos) * D + 4 * h;
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
#pragma unroll
        for (int g = 0; g < 4; ++g)
            *reinterpret_cast<float4*>(dst + db * 32 + 8 * g) =
                make_float4(acc[db][4 * g] * inv, acc[db][4 * g + 1] * inv, acc[db][4 * g + 2] * inv, acc[db][4 * g + 3] * inv);
    if (h == 0) lse[seg + qpos] = ltot > 0.f ? fmaf(log2f(ltot), LN2, m * tau) : -INFINITY;
}

template <int D, int KS, bool INDIRECT>
static int launch_f32_t(const float* q, const float* k, const float* v, const uint32_t* q_key, const uint32_t* k_key,
                        const int32_t* work, int n_work, int S, int T, float tau, int strict, float* o, float* lse,
                        const int32_t* n_keep_q, hipStream_t st)
{
    using L = F32Tiles<D, KS>;
    static std::atomic<unsigned long long> lds_allowed{0};
    const int rc = allow_dynamic_lds(reinterpret_cast<const void*>(&attn_fwd_f32_kernel<D, KS, INDIRECT>), L::SMEM, lds_allowed);
    if (rc != SCFA_OK) return rc;
    return launch_in_grids(S, n_work, L::THREADS, [&](int first, unsigned items) -> int {
        hipLaunchKernelGGL((attn_fwd_f32_kernel<D, KS, INDIRECT>), dim3(S * items), dim3(L::THREADS), L::SMEM, st, q, k, v, q_key, k_key,
                           work, n_work, first, S, T, tau, strict, o, lse, n_keep_q);
        SCFA_HIP_TRY(hipGetLastError());
        return SCFA_OK;
    });
}

// indirect: q, k, v are the tensors in original order, fetched through the positions in the sort keys
int launch_attn_fwd_f32(const float* q, const float* k, const float* v, const uint32_t* q_key,
                        const uint32_t* k_key, const int32_t* work, int n_work, int S, int T, int d,
                        float tau, int strict, float* o, float* lse, const int32_t* n_keep_q, bool indirect, hipStream_t st)
{
    ProfScope prof(SCFA_K_FWD, st);
#define SCFA_F32_LAUNCH(DD, KS)                                                                                             \
    (indirect ? launch_f32_t<DD, KS, true>(q, k, v, q_key, k_key, work, n_work, S, T, tau, strict, o, lse, n_keep_q, st)    \
              : launch_f32_t<DD, KS, false>(q, k, v, q_key, k_key, work, n_work, S, T, tau, strict, o, lse, n_keep_q, st))
    if (d == 64) return SCFA_F32_LAUNCH(64, 2);
    if (d == 128) return SCFA_F32_LAUNCH(128, 2);
#undef SCFA_F32_LAUNCH
    return SCFA_EUNSUPPORTED;
}

}  // namespace scfa
