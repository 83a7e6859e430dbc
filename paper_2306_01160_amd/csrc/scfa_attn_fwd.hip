// Forward attention over the work list, fp16 compute format, fp32 accumulation.
//
// A workgroup owns one work item: up to 128 query rows of one bucket and the range of keys
// of the same bucket that causality can let through, or all rows of a few small buckets on
// both sides (scfa_block_ranges).  Keys are walked 64 at a time; tiles the schedule proved
// mask-free come first and run without any test, the remaining tiles test bucket and
// causality at once on the rows' sort keys, bucket << 24 | original position (paper
// Sec. 3.1 / 3.2: a local mask from the index and bucket vectors).  Sort keys ascend along
// an item's keys, so a wavefront also skips a masked tile that lies entirely outside the
// key range its own 32 queries can match.
//
// A wavefront keeps its query rows in the lanes: S^T = K Q^T puts one query per lane
// (column) and 16 keys per accumulator block in its registers, so the softmax
// statistics are per-lane scalars and S^T's accumulator layout is already the
// B-operand layout of O^T += V^T P^T.  V^T comes from the row-major V tile through
// transposing LDS reads.
//
// K / V tiles and the key positions travel global memory -> LDS asynchronously (no
// registers, no LDS stores), NBUF - 1 tiles ahead of the one being computed, into a ring of
// NBUF swizzled buffers; one workgroup barrier per tile both publishes the tile that has
// landed and retires the buffer that is refilled next.
//
// The permuted queries and keys are the inputs' own values (bf16 -> fp16 is exact), so the
// contraction yields <q, k> exactly up to the fp32 accumulation, and the softmax scale enters
// as one fused multiply-add per element, p = 2^(tau log2(e) (<q, k> - m) + bias): the
// logsumexp this kernel hands out carries no rounding of the operands.  (The backward kernels
// fold the scale into their register-resident operand instead and save that instruction: a
// 2^-12 relative error per element of the recomputed scores does not matter to the gradients,
// but it would be the largest term of the logsumexp error.)
//
// Online softmax (paper App. B.1, running maximum and sum, NaN-safe for fully masked
// rows): the accumulator is un-normalised and divided by the sum once at the end.  The
// reference maximum m (of the raw sums) is only raised when some row's tile maximum exceeds
// it by more than LAZY_LOG2 base-2 units (then the accumulator and the sum are rescaled by
// 2^(c (m_old - m_new)), c = tau log2(e)); between raises P = 2^(c (s - m)) may exceed 1 but
// stays inside the fp16 range.  Once every
// row of a wavefront has a finite reference, the tile maximum is not even computed: the
// row sum of the packed probabilities, needed anyway, exceeds 2^15 in some lane whenever
// a probability has left the fp16 range (packing truncates to at most 65504), and only
// then is the tile redone with its maximum as the new reference.  Because
// m changes rarely, -m is kept splatted over an accumulator block and the score
// contraction starts from it: the matrix core delivers s - m and the only per-element
// vector work left is the scaling, the exponential, the packing and the row sum.  A row that never
// sees an allowed key keeps m = -inf and l = 0; its exponent base is 0 (the paper's
// replacement of -inf by 0), every p is 2^(-inf) = 0, and it is written as zeros with
// LSE = -inf.
#include "scfa_common.hpp"
#include "scfa_mma.hpp"
#include "scfa_rows.hpp"

#include <math.h>
#include <type_traits>

namespace scfa {

constexpr float LAZY_LOG2 = 6.0f;
constexpr float SUM_LIMIT = 32768.f;   // a lane's tile sum above this may hide a probability beyond the fp16 range

// LDS ring of the forward kernel: as many buffers as three resident workgroups allow
template <int D>
struct FwdRing {
    static constexpr int BUF_BYTES = FWD_TILE_N * D * 4 + FWD_TILE_N * 4;
    static constexpr int NBUF = D == 64 ? 3 : 2;
};

// QK-dropping: the output rows of dropped queries are zeros and their LSE is -inf.  Every workgroup of the forward kernel, the
// ones without work included, writes a strided share of its segment's dropped rows after its own stores (a launch of its own
// for them ran with nothing beside it; why after: zero_dropped_rows in scfa_attn_bwd.hip).  key_seg: the segment's query index vector, dropped positions from n_keep on.
template <int D, int THREADS>
__device__ __forceinline__ void fill_dropped_rows(const uint32_t* __restrict__ key_seg, int n_keep, int T, int w, int n_wg,
                                                  uint16_t* __restrict__ o, float* __restrict__ lse, size_t seg)
{
    constexpr int CPR = D / 8, R = THREADS / CPR;   // 16-byte pieces per bf16 row, rows per pass
    const int sub = (int)threadIdx.x / CPR, c = (int)threadIdx.x % CPR;
    for (long long r = (long long)n_keep + (long long)w * R + sub; r < T; r += (long long)n_wg * R) {
        const size_t pos = seg + (key_seg[r] & KEY_POS_MASK);
        store_stream(reinterpret_cast<uint4*>(o + pos * D) + c, make_uint4(0u, 0u, 0u, 0u));
        if (c == 0) lse[pos] = -INFINITY;
    }
}

// OWN_Q: q holds the bf16 rows in original order; the workgroup fetches its own through the positions in the sort keys,
// converts them, and writes the fp16 copy in permuted order to q_out (nullable: no backward wanted).  Otherwise q is that copy.
// KS: groups of NW wavefronts that share an item's key tiles (see split_keys), each with its own LDS ring and its own sums.
template <int D, int NW, int QB, bool OWN_Q, int KS>
__global__ __launch_bounds__(NW * KS * 64) __attribute__((amdgpu_waves_per_eu(D == 64 && KS == 1 ? 3 : 2))) void attn_fwd_f16_kernel(
    const uint16_t* __restrict__ q, const uint16_t* __restrict__ k, const uint16_t* __restrict__ v,
    const uint32_t* __restrict__ q_key, const uint32_t* __restrict__ k_key,
    const int32_t* __restrict__ work, int n_work, int first, int S, int T, float tau, int strict,
    uint16_t* __restrict__ o, float* __restrict__ lse, uint16_t* __restrict__ o_f16, const int32_t* __restrict__ n_keep_q,
    uint16_t* __restrict__ q_out)
{
    static_assert(NW * QB * 32 == FWD_TILE_M, "workgroup must cover the forward query tile");
    const float cexp = tau * LOG2E;   // scores are raw <q, k> sums; the exponent of every probability is cexp * (sum - m)
    constexpr int BN = FWD_TILE_N;
    constexpr int THREADS = NW * 64;                  // of one of the KS groups
    constexpr int NBUF = FwdRing<D>::NBUF;            // LDS ring; NBUF - 1 tiles are in flight
    constexpr int TILE_ELEMS = BN * D;
    constexpr int BUF_BYTES = FwdRing<D>::BUF_BYTES;  // K tile, V tile, key positions
    constexpr int LOADS_PER_TILE = 2 * AsyncTile<D, BN, THREADS>::ROUNDS + 1;   // per wavefront
    constexpr int KPW = BN / NW;                      // key positions loaded per wavefront
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_all[];
    const int group = KS == 1 ? 0 : __builtin_amdgcn_readfirstlane((int)threadIdx.x / THREADS);
    unsigned char* const smem_raw = smem_all + group * (NBUF * BUF_BYTES);
    auto k_tile = [&](int buf) { return reinterpret_cast<const uint16_t*>(smem_raw + buf * BUF_BYTES); };
    auto v_tile = [&](int buf) { return reinterpret_cast<const uint16_t*>(smem_raw + buf * BUF_BYTES + TILE_ELEMS * 2); };
    auto kpos_tile = [&](int buf) { return reinterpret_cast<uint32_t*>(smem_raw + buf * BUF_BYTES + TILE_ELEMS * 4); };
    const uint32_t lds0 = lds_address(smem_raw);

    int s, w;
    place_workgroup(blockIdx.x, S, s, w);
    w += first;
    const int32_t* it = work + ((size_t)s * n_work + w) * WORK_STRIDE;
    const int q_begin = it[W_QBEGIN], q_count = it[W_QCOUNT];
    const int k_begin = it[W_KBEGIN], k_count = it[W_KCOUNT], k_nomask = it[W_KNOMASK];
    const size_t seg = (size_t)s * T;
    auto fill_dropped = [&] { if (n_keep_q) fill_dropped_rows<D, THREADS * KS>(q_key + seg, n_keep_q[s], T, w, n_work, o, lse, seg); };
    if (q_count <= 0) return fill_dropped();   // no work: only the share of the dropped rows (n_keep_q: QK-dropping, else null)

    const int tid = threadIdx.x % THREADS, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, l32 = lane & 31, h = lane >> 5;

    const uint16_t* kbase = k + (seg + k_begin) * D;
    const uint16_t* vbase = v + (seg + k_begin) * D;
    const uint32_t* kib = k_key + seg + k_begin;
    const int n_tiles = (k_count + BN - 1) / BN;
    const int n_free = k_nomask / BN;            // leading tiles that need no mask

    AsyncTile<D, BN, THREADS> loader;
    loader.init();
    const u32x4 k_desc = make_desc(kbase, (uint32_t)k_count * D * 2);
    const u32x4 v_desc = make_desc(vbase, (uint32_t)k_count * D * 2);
    const u32x4 p_desc = make_desc(kib, (uint32_t)k_count * 4);
    // every wavefront issues the same number of loads per tile (BN / NW key positions each), so one
    // vmcnt threshold serves all; tiles past the end read zeros into a buffer nobody uses
    auto issue = [&](int jt, int buf) {
        const uint32_t base = lds0 + (uint32_t)(buf * BUF_BYTES);
        loader.load(k_desc, jt * loader.TILE_BYTES, base);
        loader.load(v_desc, jt * loader.TILE_BYTES, base + TILE_ELEMS * 2);
        if (lane < KPW)
            async_load4(p_desc, __builtin_amdgcn_readfirstlane(base + TILE_ELEMS * 4 + wave * KPW * 4),
                        (wave * KPW + lane) * 4, jt * BN * 4);
    };
    // the first tiles are on their way while the rows of the item are fetched and looked at: behind them they were one memory latency
    // more of every item (192 x 1024 rows in 16 buckets 160.5 -> 158.7 us a step, 36 x 8192 272 -> 268; both gradients likewise, but for dK/dV at d = 128)
#pragma unroll
    for (int u = 0; u < NBUF - 1; ++u) issue(u * KS + group, u);

    int cur = 0;
    auto refill_of = [&] { return cur == 0 ? NBUF - 1 : cur - 1; };    // the buffer of the tile before
    auto mark_end = [&](int jt) {                                      // keys past the end of a ragged tile are never allowed
        const int key = jt * BN + wave * KPW + lane;
        if (lane < KPW && key >= k_count) kpos_tile(cur)[wave * KPW + lane] = KEY_PAST_END;
    };
    // A wavefront without rows only loads (see dkdv_item).  In a loop of its own at d = 64, where the steps of the others are ordered worse with a
    // test (forward of 24 x 16384 rows in one bucket, loop / test 910 / 921 us, QK-dropping 16 x 16384 half kept 189 / 200); by a test in every
    // step at d = 128, where they are ordered better with it (1 x 65536 half kept 473 / 456, 2 x 37504 385 / 378).
    const bool idle = wave * (QB * 32) >= q_count;
    if (D == 64 && idle) {
        for (int jt = 0; jt < n_tiles; jt += KS) {
            wait_async<LOADS_PER_TILE * (NBUF - 2)>();
            mark_end(jt + group);
            lds_barrier();
            issue(jt + group + (NBUF - 1) * KS, refill_of());
            cur = cur == NBUF - 1 ? 0 : cur + 1;
        }
        wait_async<0>();
        for (int i = 0; i < KS; ++i) lds_barrier();
        return fill_dropped();
    }

    int qrow[QB], qpos[QB];
    // a key is allowed iff (its sort key - qlo) <= qspan: same bucket, position <= the query's (< if strict)
    uint32_t qlo[QB], qspan[QB];
    bool qvalid[QB];
    f16x8 qf[QB][D / 16];
#pragma unroll
    for (int b = 0; b < QB; ++b) {
        qrow[b] = (wave * QB + b) * 32 + l32;
        qvalid[b] = qrow[b] < q_count;
        const int qr = min(qrow[b], q_count - 1);          // rows past the end repeat the last one
        const uint32_t qk_ = q_key[seg + q_begin + qr];
        const int qp_ = (int)(qk_ & KEY_POS_MASK);
        qpos[b] = qvalid[b] ? qp_ : -1;
        const bool some = qvalid[b] && qp_ - strict >= 0;
        qlo[b] = some ? (qk_ & ~KEY_POS_MASK) : KEY_NEVER;   // KEY_NEVER, span 0: every key is masked
        qspan[b] = some ? (uint32_t)(qp_ - strict) : 0u;
        const uint16_t* qp = q + (seg + (OWN_Q ? qp_ : q_begin + qr)) * D + h * 8;
#pragma unroll
        for (int kk = 0; kk < D / 16; ++kk) {
            uint4 x = *reinterpret_cast<const uint4*>(qp + kk * 16);
            if (OWN_Q) x = convert_chunk<1>(x, 1.f);
            qf[b][kk] = as_f16x8(x);
        }
    }
#pragma unroll
    for (int b = 0; b < QB; ++b)
#pragma unroll
        for (int kk = 0; kk < D / 16; ++kk) touch(qf[b][kk]);   // loaded before the tile loop starts

    f32x16 oacc[QB][D / 32];
    f32x16 start[QB];                // -(finite reference maximum), in all 16 registers
    float m[QB], thr[QB], lsum[QB];  // reference maximum (raw <q, k> units), raise threshold on s - m, partial row sum
#pragma unroll
    for (int b = 0; b < QB; ++b) {
#pragma unroll
        for (int db = 0; db < D / 32; ++db) oacc[b][db] = zero16();
#pragma unroll
        for (int i = 0; i < 16; ++i) start[b][i] = 0.f;
        m[b] = -INFINITY; thr[b] = -INFINITY; lsum[b] = 0.f;   // the first finite score always raises
    }

    // the sort keys any query of this wavefront may attend to lie in [qlo_wave, qhi_wave]
    uint32_t qlo_wave = 0xffffffffu, qhi_wave = 0u;
#pragma unroll
    for (int b = 0; b < QB; ++b)
        if (qlo[b] != KEY_NEVER) { qlo_wave = min(qlo_wave, qlo[b]); qhi_wave = max(qhi_wave, qlo[b] + qspan[b]); }
    qlo_wave = __builtin_amdgcn_readfirstlane(wave_reduce(qlo_wave, min_u32));
    qhi_wave = __builtin_amdgcn_readfirstlane(wave_reduce(qhi_wave, max_u32));

    // lane-invariant offsets of the transposing V reads
    int v_off[4][D / 32][2];
#pragma unroll
    for (int c4 = 0; c4 < 4; ++c4)
#pragma unroll
        for (int db = 0; db < D / 32; ++db) swz_trans_offsets<D>(c4 * 16, db * 32, lane, v_off[c4][db][0], v_off[c4][db][1]);

    bool settled = false;   // every row of this wavefront has a finite reference maximum (wave-uniform)
    auto tile = [&](int buf, auto masked_tag) {
        constexpr bool MASKED = decltype(masked_tag)::value;
        const uint16_t* Kt = k_tile(buf);
        const uint16_t* Vt = v_tile(buf);
        const uint32_t* kpos_t = kpos_tile(buf);
        // S^T = K Q^T - m : [key block kb][query block b]
        f32x16 sacc[2][QB];
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
            for (int b = 0; b < QB; ++b) sacc[kb][b] = start[b];
        if (D == 128) {
            // two wavefronts per SIMD do not hide the LDS latency of a read issued at its use: the K row
            // fragments of a contraction step are requested one step ahead
            f16x8 fk[2][2];
            fk[0][0] = swz_rows<D>(Kt, l32, h * 8);
            fk[0][1] = swz_rows<D>(Kt, 32 + l32, h * 8);
#pragma unroll
            for (int kk = 0; kk < D / 16; ++kk) {
                if (kk + 1 < D / 16) {
                    fk[(kk + 1) & 1][0] = swz_rows<D>(Kt, l32, (kk + 1) * 16 + h * 8);
                    fk[(kk + 1) & 1][1] = swz_rows<D>(Kt, 32 + l32, (kk + 1) * 16 + h * 8);
                }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                    for (int b = 0; b < QB; ++b) sacc[kb][b] = mfma16(fk[kk & 1][kb], qf[b][kk], sacc[kb][b]);
                __builtin_amdgcn_sched_barrier(0);
            }
        } else {
#pragma unroll
            for (int kk = 0; kk < D / 16; ++kk)
#pragma unroll
                for (int kb = 0; kb < 2; ++kb) {
                    const f16x8 a = swz_rows<D>(Kt, kb * 32 + l32, kk * 16 + h * 8);
#pragma unroll
                    for (int b = 0; b < QB; ++b) sacc[kb][b] = mfma16(a, qf[b][kk], sacc[kb][b]);
                }
        }

        if (MASKED) {   // bucket and causal test in one range test on the sort keys
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const uint4 kp = *reinterpret_cast<const uint4*>(&kpos_t[kb * 32 + 8 * g + 4 * h]);
#pragma unroll
                    for (int b = 0; b < QB; ++b) {
                        if (kp.x - qlo[b] > qspan[b]) sacc[kb][b][4 * g + 0] = -INFINITY;
                        if (kp.y - qlo[b] > qspan[b]) sacc[kb][b][4 * g + 1] = -INFINITY;
                        if (kp.z - qlo[b] > qspan[b]) sacc[kb][b][4 * g + 2] = -INFINITY;
                        if (kp.w - qlo[b] > qspan[b]) sacc[kb][b][4 * g + 3] = -INFINITY;
                    }
                }
        }

        // lane-local tile maximum per query; raise the reference only when needed
        auto raise_ref = [&]() {
        float mx[QB];
        bool raise = false;
#pragma unroll
        for (int b = 0; b < QB; ++b) {
            float a0 = sacc[0][b][0], a1 = sacc[1][b][0];
#pragma unroll
            for (int i = 1; i < 16; i += 2) {
                a0 = fmaxf(a0, fmaxf(sacc[0][b][i], sacc[0][b][(i + 1) & 15]));
                a1 = fmaxf(a1, fmaxf(sacc[1][b][i], sacc[1][b][(i + 1) & 15]));
            }
            mx[b] = fmaxf(a0, a1);
            raise |= mx[b] > thr[b];                    // -inf > -inf is false: no NaN is ever formed
        }
        if (__ballot(raise) != 0ull) {
#pragma unroll
            for (int b = 0; b < QB; ++b) {
                const float st_old = start[b][0];
                const float m_new = fmaxf(m[b], half_max(mx[b]) - st_old);   // tile maximum back in score units
                const float m_use = m_new == -INFINITY ? 0.f : m_new;
                float alpha = fast_exp2((m[b] - m_use) * cexp);                       // m = -inf -> 0
                asm volatile("" : "+v"(alpha));   // rare path: keeps the rescale from being speculated
                lsum[b] *= alpha;
#pragma unroll
                for (int db = 0; db < D / 32; ++db)
#pragma unroll
                    for (int i = 0; i < 16; ++i) oacc[b][db][i] *= alpha;
                const float st_new = -m_use;
                const float shift = st_new - st_old;    // scores of this tile move to the new reference
#pragma unroll
                for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                    for (int i = 0; i < 16; ++i) sacc[kb][b][i] += shift;
#pragma unroll
                for (int i = 0; i < 16; ++i) start[b][i] = st_new;
                m[b] = m_new;
                thr[b] = m_new == -INFINITY ? -INFINITY : LAZY_LOG2 / cexp;
            }
        }
        };

        // P = 2^(c (s - m) + bias), packed to fp16 (truncating: at most 65504, never inf); row sums from the
        // packed values
        f16x8 pf[QB][4];
        float lt[QB];
        auto exp_pack = [&]() {
#pragma unroll
        for (int b = 0; b < QB; ++b) {
            float l0 = 0.f, l1 = 0.f;
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int cc = 0; cc < 2; ++cc) {
                    uint32_t wv[4];
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const float p0 = fast_exp2(fmaf(sacc[kb][b][8 * cc + 2 * j], cexp, RTZ_BIAS_LOG2));
                        const float p1 = fast_exp2(fmaf(sacc[kb][b][8 * cc + 2 * j + 1], cexp, RTZ_BIAS_LOG2));
                        wv[j] = pack_f16(p0, p1);
                    }
                    l0 = add_pair(wv[0], l0); l1 = add_pair(wv[1], l1);
                    l0 = add_pair(wv[2], l0); l1 = add_pair(wv[3], l1);
                    pf[b][kb * 2 + cc] = as_f16x8(make_uint4(wv[0], wv[1], wv[2], wv[3]));
                }
            lt[b] = l0 + l1;
        }
        };

        // Until every row of the wavefront has a finite reference the tile maximum is taken first.
        // After that the maximum is not computed at all: the sum of the packed probabilities,
        // which is needed anyway, tells whether any of them left the fp16 range (a probability
        // beyond 2^15 makes its lane's sum exceed 2^15), and only then is the tile redone with
        // its maximum as the new reference.
        // (d = 64 only: at d = 128 the matrix cores, not the vector units, set the pace, and keeping
        // the scores alive for a possible second pass costs more than the maxima it saves)
        const bool by_sum = D == 64 && settled;
        if (!by_sum) {
            raise_ref();
            bool unset = false;
#pragma unroll
            for (int b = 0; b < QB; ++b) unset |= thr[b] == -INFINITY;
            settled = __ballot(unset) == 0ull;
        }
        exp_pack();
        if (by_sum) {
            bool big = false;
#pragma unroll
            for (int b = 0; b < QB; ++b) big |= lt[b] > SUM_LIMIT;
            if (__ballot(big) != 0ull) { raise_ref(); exp_pack(); }
        }
#pragma unroll
        for (int b = 0; b < QB; ++b) lsum[b] += lt[b];

        // O^T += V^T P^T
        if (D == 128) {   // the V^T fragments of a 16-key chunk are requested while the previous chunk's products run
            f16x8 fv[2][D / 32];
#pragma unroll
            for (int db = 0; db < D / 32; ++db) fv[0][db] = swz_trans(Vt, v_off[0][db][0], v_off[0][db][1]);
#pragma unroll
            for (int c4 = 0; c4 < 4; ++c4) {
                if (c4 + 1 < 4) {
#pragma unroll
                    for (int db = 0; db < D / 32; ++db) fv[(c4 + 1) & 1][db] = swz_trans(Vt, v_off[c4 + 1][db][0], v_off[c4 + 1][db][1]);
                }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int db = 0; db < D / 32; ++db)
#pragma unroll
                    for (int b = 0; b < QB; ++b) oacc[b][db] = mfma16(fv[c4 & 1][db], pf[b][c4], oacc[b][db]);
                __builtin_amdgcn_sched_barrier(0);
            }
        } else {
#pragma unroll
            for (int c4 = 0; c4 < 4; ++c4)
#pragma unroll
                for (int db = 0; db < D / 32; ++db) {
                    const f16x8 a = swz_trans(Vt, v_off[c4][db][0], v_off[c4][db][1]);
#pragma unroll
                    for (int b = 0; b < QB; ++b) oacc[b][db] = mfma16(a, pf[b][c4], oacc[b][db]);
                }
        }
    };

    // one step: wait for this wavefront's share of tile jt, mark keys past the end of a ragged
    // tile (always a masked tile), barrier, refill the buffer everyone has just left, compute.
    // With KS groups group g takes tiles g, g + KS, ..., all of them the same number of steps (the barrier is the workgroup's):
    // a tile past the end is all KEY_PAST_END and skipped.
    auto step = [&](int jt, auto masked_tag) {
        constexpr bool MASKED = decltype(masked_tag)::value;
        wait_async<LOADS_PER_TILE * (NBUF - 2)>();
        if (MASKED) mark_end(jt);
        lds_barrier();
        issue(jt + (NBUF - 1) * KS, refill_of());
        // sort keys ascend along the keys of an item: a tile that lies entirely above or entirely
        // below what the queries of this wavefront may attend to contributes nothing to it
        bool skip = D == 128 && idle;
        if (MASKED && !skip)
            skip = (uint32_t)__builtin_amdgcn_readfirstlane(kpos_tile(cur)[0]) > qhi_wave ||
                   (uint32_t)__builtin_amdgcn_readfirstlane(kpos_tile(cur)[BN - 1]) < qlo_wave;
        if (!skip) tile(cur, masked_tag);
        cur = cur == NBUF - 1 ? 0 : cur + 1;
    };
    int jt = 0;
    for (; jt + KS <= n_free; jt += KS) step(jt + group, std::false_type{});
    for (; jt < n_tiles; jt += KS) step(jt + group, std::true_type{});
    wait_async<0>();   // nothing may still be landing in LDS when the wavefront ends
    lds_barrier();     // ... nor anyone be reading it: it carries the results out

    if constexpr (KS == 2) {   // the second group's sums join the first's, both brought to the larger reference
        static_assert(QB == 1, "one block of queries per wavefront");
        using Stage = AccStage<D / 32>;
        static_assert(NW * (RowStage<D * 2>::BYTES + Stage::BYTES + 512) <= KS * NBUF * BUF_BYTES, "LDS of the merge");
        unsigned char* const at = smem_all + NW * RowStage<D * 2>::BYTES + wave * (Stage::BYTES + 512);
        const Stage acc{at};
        float* const ml = reinterpret_cast<float*>(at + Stage::BYTES);
        if (group == 1) {
#pragma unroll
            for (int db = 0; db < D / 32; ++db) acc.put(db, oacc[0][db], lane);
            ml[lane] = m[0];
            ml[64 + lane] = lsum[0];
        }
        lds_barrier();
        if (group == 1) return fill_dropped();
        const float m_other = ml[lane], m_new = fmaxf(m[0], m_other), m_use = m_new == -INFINITY ? 0.f : m_new;
        const float mine = fast_exp2((m[0] - m_use) * cexp), theirs = fast_exp2((m_other - m_use) * cexp);   // -inf: 0
        lsum[0] = fmaf(lsum[0], mine, ml[64 + lane] * theirs);
#pragma unroll
        for (int db = 0; db < D / 32; ++db) acc.merge(db, oacc[0][db], mine, theirs, lane);
        m[0] = m_new;
    }

    RowStage<D * 2> stage{smem_all + wave * RowStage<D * 2>::BYTES};
#pragma unroll
    for (int b = 0; b < QB; ++b) {
        const int n_rows = q_count - (wave * QB + b) * 32;     // valid rows of this block
        const float ltot = half_sum(lsum[b]);
        const float inv = ltot > 0.f ? 1.f / ltot : 0.f;
        if (h == 0 && qvalid[b]) lse[seg + qpos[b]] = ltot > 0.f ? (m[b] * cexp + log2f(ltot)) * LN2 : -INFINITY;
        auto original = [&](int row) { return seg + (size_t)__shfl(qpos[b], row); };
#pragma unroll
        for (int db = 0; db < D / 32; ++db)
#pragma unroll
            for (int i = 0; i < 16; ++i) oacc[b][db][i] *= inv;
#pragma unroll
        for (int db = 0; db < D / 32; ++db)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                uint2 pk;
                const __bf16 y0 = (__bf16)oacc[b][db][4 * g + 0], y1 = (__bf16)oacc[b][db][4 * g + 1];
                const __bf16 y2 = (__bf16)oacc[b][db][4 * g + 2], y3 = (__bf16)oacc[b][db][4 * g + 3];
                pk.x = (uint32_t)__builtin_bit_cast(uint16_t, y0) | ((uint32_t)__builtin_bit_cast(uint16_t, y1) << 16);
                pk.y = (uint32_t)__builtin_bit_cast(uint16_t, y2) | ((uint32_t)__builtin_bit_cast(uint16_t, y3) << 16);
                reinterpret_cast<uint2*>(stage.chunk(l32, db * 4 + g))[h] = pk;
            }
        stage.template store<true>(o, n_rows, lane, original);
        if (o_f16) {   // the same values with 11 significant bits, for the backward's D = <dO, O>
#pragma unroll
            for (int db = 0; db < D / 32; ++db)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    uint2 hk;
                    const _Float16 z0 = (_Float16)oacc[b][db][4 * g + 0], z1 = (_Float16)oacc[b][db][4 * g + 1];
                    const _Float16 z2 = (_Float16)oacc[b][db][4 * g + 2], z3 = (_Float16)oacc[b][db][4 * g + 3];
                    hk.x = (uint32_t)__builtin_bit_cast(uint16_t, z0) | ((uint32_t)__builtin_bit_cast(uint16_t, z1) << 16);
                    hk.y = (uint32_t)__builtin_bit_cast(uint16_t, z2) | ((uint32_t)__builtin_bit_cast(uint16_t, z3) << 16);
                    reinterpret_cast<uint2*>(stage.chunk(l32, db * 4 + g))[h] = hk;
                }
            stage.template store<false>(o_f16, n_rows, lane, original);
        }
        if (OWN_Q && q_out) {
#pragma unroll
            for (int kk = 0; kk < D / 16; ++kk)
                *reinterpret_cast<uint4*>(stage.chunk(l32, 2 * kk + h)) = __builtin_bit_cast(uint4, qf[b][kk]);
            stage.template store<false>(q_out, n_rows, lane, [&](int row) { return seg + (size_t)(q_begin + (wave * QB + b) * 32 + row); });
        }
    }
    fill_dropped();
}

// Whether two groups of wavefronts share the key tiles of an item.  A launch that cannot give every CU two or three workgroups is
// as long as its longest item, a bucket's rows over 64 tiles by one wavefront per SIMD; with the tiles shared the other half of
// the SIMD's registers works on the same item.  Where the CUs are full without it, it only adds the merge and takes the third
// wavefront per SIMD away (d = 64).  Forward call in us, one group / two groups, d = 64 (d = 128 gains the same or more):
//   128 items  rows of 1024: 33.9 / 31.2   4096: 78 / 69    16384: 223 / 183    (556 rows, 117 items: 31.3 / 30.1)
//   256 items  rows of 512: 31.1 / 33.4    1024: 38.9 / 37.7   2048: 44.6 / 39.7   8192: 123 / 104
//   384 items  rows of 1024: 44.1 / 43.7   8192: 131 / 106     16384: 236 / 189
//   512 items  rows of 1024: 39.8 / 45.5   2048: 49.9 / 47.1   4096: 81 / 71     (8 buckets of 8192, one dispatched after the
//   other: 175 / 179)                      768 items, rows of 8192: 161 / 177
// QK-dropping, whose counts the host does not know, is taken as half kept: 32 x 2048 36.6 / 33.4, 12 x 8192 85.6 / 69.4 (with 0.9
// kept 51.4 / 49.2 and 142 / 146, with 0.2 25.0 / 24.0).
static bool split_keys(int S, int T, int nb, bool drop)
{
    const long long items = (long long)S * T / (drop ? 2 * FWD_TILE_M : FWD_TILE_M), rows = drop ? T / 2 : T / nb;
    return rows >= 512 && items <= rows / 4 && items <= (nb <= 2 && !drop ? 512 : 384);
}

template <int D, bool OWN_Q, int KS>
static int launch_fwd_t(const void* q, const void* k, const void* v, const uint32_t* q_key, const uint32_t* k_key,
                        const int32_t* work, int n_work, int S, int T, float tau, int strict, void* o,
                        float* lse, void* o_f16, const int32_t* n_keep_q, void* q_out, hipStream_t st)
{
    constexpr size_t smem = (size_t)KS * FwdRing<D>::NBUF * FwdRing<D>::BUF_BYTES;
    static std::atomic<unsigned long long> lds_allowed{0};
    { const int rc_ = allow_dynamic_lds(reinterpret_cast<const void*>(&attn_fwd_f16_kernel<D, 4, 1, OWN_Q, KS>), (int)smem, lds_allowed); if (rc_ != SCFA_OK) return rc_; }
    return launch_in_grids(S, n_work, 256 * KS, [&](int first, unsigned items) -> int {
        hipLaunchKernelGGL((attn_fwd_f16_kernel<D, 4, 1, OWN_Q, KS>), dim3(S * items), dim3(256 * KS), smem, st, (const uint16_t*)q,
                           (const uint16_t*)k, (const uint16_t*)v, q_key, k_key, work, n_work, first, S, T, tau,
                           strict, (uint16_t*)o, lse, (uint16_t*)o_f16, n_keep_q, (uint16_t*)q_out);
        SCFA_HIP_TRY(hipGetLastError());
        return SCFA_OK;
    });
}

// workgroups of the forward kernel one CU holds at once (registers, LDS ring)
int occupancy_attn_fwd_bf16(int d, int* out)
{
    if (d == 64) {
        constexpr size_t smem = (size_t)FwdRing<64>::NBUF * FwdRing<64>::BUF_BYTES;
        SCFA_HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(&attn_fwd_f16_kernel<64, 4, 1, false, 1>), hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem));
        SCFA_HIP_TRY(hipOccupancyMaxActiveBlocksPerMultiprocessor(out, reinterpret_cast<const void*>(&attn_fwd_f16_kernel<64, 4, 1, false, 1>), 256, smem));
        return SCFA_OK;
    }
    if (d == 128) {
        constexpr size_t smem = (size_t)FwdRing<128>::NBUF * FwdRing<128>::BUF_BYTES;
        SCFA_HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(&attn_fwd_f16_kernel<128, 4, 1, false, 1>), hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem));
        SCFA_HIP_TRY(hipOccupancyMaxActiveBlocksPerMultiprocessor(out, reinterpret_cast<const void*>(&attn_fwd_f16_kernel<128, 4, 1, false, 1>), 256, smem));
        return SCFA_OK;
    }
    return SCFA_EUNSUPPORTED;
}

int launch_attn_fwd_bf16(const void* q, const void* k, const void* v, const uint32_t* q_key,
                         const uint32_t* k_key, const int32_t* work, int n_work, int S, int T, int d,
                         float tau, int strict, void* o, float* lse, void* o_f16, const int32_t* n_keep_q, bool own_q, void* q_out,
                         hipStream_t st)
{
    ProfScope prof(SCFA_K_FWD, st);
    const int nb = n_work - (T + FWD_TILE_M - 1) / FWD_TILE_M;     // the list has room for ceil(T / tile) + nb items, unless the caller cut it
    const bool split = split_keys(S, T, nb < 1 ? 1 : nb, n_keep_q != nullptr);
#define SCFA_FWD_LAUNCH_(DD, KS)                                                                                                      \
    (own_q ? launch_fwd_t<DD, true, KS>(q, k, v, q_key, k_key, work, n_work, S, T, tau, strict, o, lse, o_f16, n_keep_q, q_out, st)  \
           : launch_fwd_t<DD, false, KS>(q, k, v, q_key, k_key, work, n_work, S, T, tau, strict, o, lse, o_f16, n_keep_q, nullptr, st))
#define SCFA_FWD_LAUNCH(DD) (split ? SCFA_FWD_LAUNCH_(DD, 2) : SCFA_FWD_LAUNCH_(DD, 1))
    if (d == 64) return SCFA_FWD_LAUNCH(64);
    if (d == 128) return SCFA_FWD_LAUNCH(128);
#undef SCFA_FWD_LAUNCH_
#undef SCFA_FWD_LAUNCH
    return SCFA_EUNSUPPORTED;
}

}  // namespace scfa
