// Tile-skip schedule (paper Sec. 3.1: j_stop from the key / query index vectors;
// Sec. 3.2: j_start, j_stop from the bucket ids, then the causal refinement).
//
// The paper's kernels scan blocks of the index vectors inside every program.  Here
// the schedule is a pass of its own, and because this library owns the tiling it
// anchors tiles at bucket boundaries: a work item is a tile of query rows of ONE
// bucket together with the range of keys of the same bucket that the causal test
// can let through.  Positions are increasing inside a bucket (stable sort), so both
// range ends are binary searches in the key (query) index vector:
//   forward item : keys with position <= largest query position of the tile
//                  (and the prefix with position <= smallest query position needs no mask)
//   backward item: queries with position >= smallest key position of the tile
//                  (only those with position < largest key position need a mask)
// Buckets with fewer rows than a tile would leave most of every tile empty, so consecutive small
// buckets are put together: as many whole buckets as fit one tile of the tiled side form one
// item that spans all their rows on both sides (build_list says how small).  The kernels tell the buckets of such an item
// apart by the sort keys (bucket << 24 | position), which they test in every tile of it.
// Items of a segment are emitted bucket pair by bucket pair, and inside a pair in order of
// decreasing work.  Workgroups that run at the same time then share the keys / values
// (forward) or queries / dO rows (backward) of one or two buckets, which stay in the L2 of
// their XCD (measured at 8 buckets of 2048: 0.15-0.2 GB fetched from memory per attention
// kernel instead of 0.6 GB with a purely work-ordered list), while the last workgroups of a
// launch are still the short items.
//
// One workgroup builds one list of one segment (the forward and the backward list are
// independent).  The index vector that is searched is first copied into LDS when it fits,
// so the dependent steps of the binary searches cost LDS, not global-memory, latency; when it
// does not fit, every 2^shift-th entry is copied and a search ends with <= shift steps in global
// memory.
#include "scfa_common.hpp"
#include "scfa_lists.hpp"
#include "scfa_rows.hpp"

namespace scfa {

constexpr int RANGES_THREADS = 512;

struct RangesArgs {
    int variant;
    const int32_t *q_idx, *k_idx, *q_off, *k_off;
    int T, nb, fwd_m, fwd_n, bwd_n, bwd_m, n_fwd, n_bwd, stage_shift, strict;
    int32_t *fwd_work, *bwd_work;
    long long* counters;
};

// one list (forward or backward) of segment s, by a workgroup of RANGES_THREADS
__device__ void ranges_block(const RangesArgs& ar, int s, bool backward, int32_t* smem)
{
    const int T = ar.T, nb = ar.nb, stage_shift = ar.stage_shift;
    const int32_t* __restrict__ q_off_g = ar.q_off;
    const int32_t* __restrict__ k_off_g = ar.k_off;
    const int fwd_m = ar.fwd_m, fwd_n = ar.fwd_n, bwd_n = ar.bwd_n, bwd_m = ar.bwd_m, n_fwd = ar.n_fwd, n_bwd = ar.n_bwd;
    int32_t* s_qoff = smem;                   // [nb+1]
    int32_t* s_koff = s_qoff + nb + 1;        // [nb+1]
    int32_t* s_tile_base = s_koff + nb + 1;   // [nb+1]
    int32_t* s_unit_first = s_tile_base + nb + 1;   // [nb+1]
    const int n_max_items = n_fwd > n_bwd ? n_fwd : n_bwd;
    int32_t* s_cost = s_unit_first + nb + 1;  // [max(n_fwd, n_bwd)]
    int32_t* s_idx = smem + ((4 * (nb + 1) + n_max_items + 3) & ~3);   // [T] when staged, 16-byte aligned
    if (ar.variant == SCFA_QKDROP) {
        if (threadIdx.x == 0) {
            s_qoff[0] = 0; s_qoff[1] = min(max(q_off_g[s], 0), T);
            s_koff[0] = 0; s_koff[1] = min(max(k_off_g[s], 0), T);
        }
    } else {
        for (int b = threadIdx.x; b <= nb; b += RANGES_THREADS) {
            s_qoff[b] = q_off_g[(size_t)s * (nb + 1) + b];
            s_koff[b] = k_off_g[(size_t)s * (nb + 1) + b];
        }
    }
    const int32_t* qi = ar.q_idx + (size_t)s * T;
    const int32_t* ki = ar.k_idx + (size_t)s * T;
    const int32_t* searched_g = backward ? qi : ki;    // the ranged side
    if (stage_shift == 0) {   // 16-byte loads, eight in flight per thread (the segment base is 16-byte aligned when T % 4 == 0)
        if ((T & 3) == 0) {
            const int4* src4 = reinterpret_cast<const int4*>(searched_g);
            int4* dst4 = reinterpret_cast<int4*>(s_idx);
            const int n4 = T >> 2;
            for (int t0 = 0; t0 < n4; t0 += RANGES_THREADS * 8) {
                int4 v[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const int t = t0 + u * RANGES_THREADS + threadIdx.x;
                    v[u] = t < n4 ? src4[t] : make_int4(0, 0, 0, 0);
                }
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const int t = t0 + u * RANGES_THREADS + threadIdx.x;
                    if (t < n4) dst4[t] = v[u];
                }
            }
        } else {
            for (int t = threadIdx.x; t < T; t += RANGES_THREADS) s_idx[t] = searched_g[t];
        }
    } else {                  // every 2^shift-th entry
        const int n_s = ((T - 1) >> stage_shift) + 1;
        for (int i0 = 0; i0 < n_s; i0 += RANGES_THREADS * 8) {   // eight loads in flight per thread
            int32_t v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int i = i0 + u * RANGES_THREADS + threadIdx.x;
                v[u] = i < n_s ? searched_g[(size_t)i << stage_shift] : 0;
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int i = i0 + u * RANGES_THREADS + threadIdx.x;
                if (i < n_s) s_idx[i] = v[u];
            }
        }
    }
    const Searched searched{searched_g, s_idx, stage_shift};
    __syncthreads();
    long long* cnt = ar.counters ? ar.counters + (size_t)s * 4 : nullptr;
    if (!backward && !ar.bwd_work && cnt && threadIdx.x == 0) { cnt[2] = 0; cnt[3] = 0; }
    build_list<RANGES_THREADS>(!backward, ar.strict, backward ? ki : qi, searched, backward ? s_koff : s_qoff, backward ? s_qoff : s_koff, nb,
                               backward ? bwd_n : fwd_m, backward ? bwd_m : fwd_n, backward ? n_bwd : n_fwd,
                               backward ? ar.bwd_work + (size_t)s * n_bwd * WORK_STRIDE : ar.fwd_work + (size_t)s * n_fwd * WORK_STRIDE,
                               cnt ? cnt + (backward ? 2 : 0) : nullptr, s_tile_base, s_unit_first, s_cost);
}


__global__ __launch_bounds__(RANGES_THREADS) void block_ranges_kernel(RangesArgs ar)
{
    extern __shared__ int32_t smem[];
    ranges_block(ar, blockIdx.x, blockIdx.y == 1, smem);
}

constexpr int GATHER_PER_THREAD = 4;   // 16-byte chunks per thread of the gather

// The gather of Q, K and V with the work lists beside it: both follow the sort and neither needs the other.  Workgroups
// [0, n_lists) build a list each; they are latency-bound (6 - 16 us) on a few CUs and as a launch of their own left the rest of
// the chip idle.  The others gather, GATHER_PER_THREAD chunks in flight per thread: with one, the many short workgroups with
// the lists' LDS attached took 60 us for 48 segments of 8192 rows (d = 64) where the gather alone took 53 and the lists 12;
// with four the launch takes 50 us, lists included (2 x 150 MB moved: 6.0 TB/s).
template <int MODE, bool STREAM>
__global__ __launch_bounds__(RANGES_THREADS) void gather_and_ranges_kernel(RangesArgs ar, GatherBatch batch, int S, int n_lists,
                                                                            int blocks_per_segment, int chunks_per_row)
{
    extern __shared__ int32_t smem[];
    if ((int)blockIdx.x < n_lists) {
        ranges_block(ar, blockIdx.x % S, (int)blockIdx.x >= S, smem);
        return;
    }
    const int g = blockIdx.x - n_lists;
    const int x = g % blocks_per_segment, ts = g / blocks_per_segment;
    gather_chunks<MODE, GATHER_PER_THREAD, STREAM>(batch.p[ts / S], ts % S, (long long)x * RANGES_THREADS * GATHER_PER_THREAD + threadIdx.x,
                                           RANGES_THREADS, ar.T, chunks_per_row, (int32_t)KEY_POS_MASK);
}

// ---- sort, work lists and gather in one launch, for segments whose sort keys fit LDS twice ---------------------------------
// As launches of their own they are chains of memory latencies with a launch between them: a forward of 2 x 512 rows takes 18.2 us
// with them and 14.8 with this.  Here every workgroup sorts the whole segment for itself, queries on one half of its wavefronts and keys
// on the other, into LDS, and then does its part: a list, or rows of the gather; each also writes its share of the sort keys.
constexpr int PREPARE_THREADS = 1024;
constexpr int PREPARE_WAVES = PREPARE_THREADS / 128;     // wavefronts per sorted side
constexpr int PREPARE_MAX_T = 4096;
constexpr int PREPARE_STEPS = PREPARE_MAX_T / (64 * PREPARE_WAVES);   // 64-token steps of a wavefront

struct PrepareArgs {
    const void *label_q, *label_k;
    uint32_t *q_key, *k_key;
    int32_t *q_off, *k_off;
    const uint4 *x[3];       // K, V, Q (null: the forward kernel fetches its own)
    uint4* out[3];
    int S, T, nb, nbits, strict, n_lists, n_parts, rows_per_part, fwd_m, fwd_n, n_fwd, n_bwd;
    int32_t *fwd_work, *bwd_work;
    long long* counters;
};

// LDS: both sides' sort keys, their histograms, the lists' scratch (T = 4096, 256 buckets: 54 KiB)
static size_t prepare_smem(int T, int nb_sort, int n_max)
{
    return sizeof(int32_t) * (2 * (size_t)T + 2 * (size_t)PREPARE_WAVES * nb_sort + 4 * (size_t)(nb_sort + 1) + (size_t)n_max);
}

// grid: S segments x (n_lists + n_parts), the lists of all segments first.  CPR: 16-byte chunks per row (0: nothing to gather)
template <bool DROP, bool TWO, int MODE, int CPR>
__global__ __launch_bounds__(PREPARE_THREADS) void prepare_kernel(PrepareArgs ar)
{
    extern __shared__ int32_t smem[];
    const int T = ar.T, nb = DROP ? 1 : ar.nb, nb_sort = DROP ? 2 : ar.nb;
    const int s = blockIdx.x % ar.S, part = blockIdx.x / ar.S, n_roles = ar.n_lists + ar.n_parts;
    const size_t seg = (size_t)s * T;
    uint32_t* s_qkey = reinterpret_cast<uint32_t*>(smem);
    uint32_t* s_kkey = s_qkey + T;
    int32_t* s_hist = smem + 2 * T;
    int32_t* s_qoff = s_hist + 2 * PREPARE_WAVES * nb_sort;
    int32_t* s_koff = s_qoff + nb_sort + 1;
    int32_t* s_tile_base = s_koff + nb_sort + 1;
    int32_t* s_unit_first = s_tile_base + nb_sort + 1;
    int32_t* s_cost = s_unit_first + nb_sort + 1;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = threadIdx.x & 63;
    const bool key_side = wave >= PREPARE_WAVES;
    sort_side<PREPARE_WAVES, PREPARE_STEPS, DROP, TWO>(key_side ? ar.label_k : ar.label_q, seg, T, nb_sort, ar.nbits, key_side ? wave - PREPARE_WAVES : wave, lane,
                    s_hist + (key_side ? PREPARE_WAVES * nb_sort : 0), key_side ? s_koff : s_qoff, key_side ? s_kkey : s_qkey);
    {   // this workgroup's share of the sort keys
        const int share = (T + n_roles - 1) / n_roles, t1 = min(T, (part + 1) * share);
        for (int t = part * share + (int)threadIdx.x; t < t1; t += PREPARE_THREADS) {
            ar.q_key[seg + t] = s_qkey[t];
            ar.k_key[seg + t] = s_kkey[t];
        }
    }
    if (part == 0) {
        if (DROP) {
            if (threadIdx.x == 0) { ar.q_off[s] = s_qoff[1]; ar.k_off[s] = s_koff[1]; }
        } else {
            for (int b = threadIdx.x; b <= nb; b += PREPARE_THREADS) {
                ar.q_off[(size_t)s * (nb + 1) + b] = s_qoff[b];
                ar.k_off[(size_t)s * (nb + 1) + b] = s_koff[b];
            }
        }
    }
    if (part < ar.n_lists) {
        const int32_t *qi = reinterpret_cast<const int32_t*>(s_qkey), *ki = reinterpret_cast<const int32_t*>(s_kkey);
        const bool fwd = part == 0;
        long long* cnt = ar.counters + (size_t)s * 4;
        if (ar.n_lists == 1 && threadIdx.x == 0) { cnt[2] = 0; cnt[3] = 0; }
        build_list<PREPARE_THREADS>(fwd, ar.strict, fwd ? qi : ki, Searched{fwd ? ki : qi, fwd ? ki : qi, 0}, fwd ? s_qoff : s_koff, fwd ? s_koff : s_qoff,
                                    nb, fwd ? ar.fwd_m : BWD_TILE_N, fwd ? ar.fwd_n : BWD_TILE_M, fwd ? ar.n_fwd : ar.n_bwd,
                                    fwd ? ar.fwd_work + (size_t)s * ar.n_fwd * WORK_STRIDE : ar.bwd_work + (size_t)s * ar.n_bwd * WORK_STRIDE,
                                    cnt + (fwd ? 0 : 2), s_tile_base, s_unit_first, s_cost);
        return;
    }
    if constexpr (CPR > 0) {
        constexpr int RPP = PREPARE_THREADS / CPR, N = 2;     // rows per pass; passes in flight
        const int n_k = DROP ? s_koff[1] : T, n_q = DROP ? s_qoff[1] : T;
        const int row0 = (part - ar.n_lists) * ar.rows_per_part, row1 = min(T, row0 + ar.rows_per_part);
        const int sub = (int)threadIdx.x / CPR, c = (int)threadIdx.x % CPR;
        const int n_tensors = ar.x[2] ? 3 : 2;
        for (int r0 = row0 + sub; r0 < row1; r0 += N * RPP) {
            uint4 v[3][N];
#pragma unroll
            for (int i = 0; i < 3; ++i)
#pragma unroll
                for (int j = 0; j < N; ++j) {
                    const int r = r0 + j * RPP;
                    if (i < n_tensors && r < row1 && r < (i < 2 ? n_k : n_q))
                        v[i][j] = ar.x[i][(seg + ((i < 2 ? s_kkey : s_qkey)[r] & KEY_POS_MASK)) * CPR + c];
                }
#pragma unroll
            for (int i = 0; i < 3; ++i)
#pragma unroll
                for (int j = 0; j < N; ++j) {
                    const int r = r0 + j * RPP;
                    if (i < n_tensors && r < row1 && r < (i < 2 ? n_k : n_q)) ar.out[i][(seg + r) * CPR + c] = convert_chunk<MODE>(v[i][j], 1.f);
                }
        }
    }
}

// Sorting a segment once per workgroup costs less than two launches and their latencies until there are so many rows that the
// launches are bound by the gather's bytes.  Forward call in us, apart / in one (d = 64, then 128):
//   2 x 512 rows 18.2 / 14.8, 19.6 / 16.6    48 x 512 21.3 / 16.3    32 x 1024 23.6 / 18.0    16 x 2048 25.9 / 20.9
//   64 x 2048 44.0 / 40.8, 68.9 / 68.3       24 x 4096 40.5 / 39.7   192 x 1024 training step 168 / 174, 96 x 2048 166 / 174
//   96 x 4096 100 / 110, 184 / 212           QK-dropping 32 x 2048 31.1 / 26.5   64 x 4096 82 / 90, 145 / 149
//   fp32 (lists only) 32 x 2048 46.4 / 44.8  16 x 4096 65.9 / 67.0
bool prepare_in_one(int S, int T) { return T <= PREPARE_MAX_T && (long long)S * T <= 131072; }

int launch_prepare(int variant, const void* label_q, const void* label_k, const void* q, const void* k, const void* v, void* q_p,
                   void* k_p, void* v_p, int dtype, int d, int S, int T, int nb, int n_fwd, int n_bwd, int strict, uint32_t* q_key,
                   uint32_t* k_key, int32_t* q_off, int32_t* k_off, int32_t* fwd_work, int32_t* bwd_work, int64_t* counters, hipStream_t st)
{
    const bool drop = variant == SCFA_QKDROP, f32 = dtype == SCFA_F32;
    PrepareArgs ar{label_q, label_k, q_key, k_key, q_off, k_off, {(const uint4*)k, (const uint4*)v, (const uint4*)q},
                   {(uint4*)k_p, (uint4*)v_p, (uint4*)q_p}, S, T, nb, 0, strict, bwd_work ? 2 : 1, 0, 0, f32 ? F32_TILE_M : FWD_TILE_M,
                   f32 ? F32_TILE_N : FWD_TILE_N, n_fwd, n_bwd, fwd_work, bwd_work, (long long*)counters};
    const int nb_sort = drop ? 2 : nb;
    while ((1 << ar.nbits) < nb_sort) ++ar.nbits;
    if (!f32) {
        ar.rows_per_part = d == 64 ? 512 : 256;     // 64 KiB a tensor; half and twice of it: the same within 2 %, or up to 20 % slower
        ar.n_parts = (T + ar.rows_per_part - 1) / ar.rows_per_part;
    }
    const size_t smem = prepare_smem(T, nb_sort, n_fwd > n_bwd ? n_fwd : n_bwd);
    const dim3 grid((unsigned)((size_t)S * (ar.n_lists + ar.n_parts))), block(PREPARE_THREADS);
    ProfScope prof(f32 ? SCFA_K_RANGES : SCFA_K_GATHER, st);
#define SCFA_PREPARE(MODE, CPR)                                                                                   \
    do {                                                                                                          \
        if (drop) hipLaunchKernelGGL((prepare_kernel<true, true, MODE, CPR>), grid, block, smem, st, ar);         \
        else if (nb <= 2) hipLaunchKernelGGL((prepare_kernel<false, true, MODE, CPR>), grid, block, smem, st, ar); \
        else hipLaunchKernelGGL((prepare_kernel<false, false, MODE, CPR>), grid, block, smem, st, ar);            \
    } while (0)
    if (f32) SCFA_PREPARE(0, 0);
    else if (dtype == SCFA_BF16 && d == 64) SCFA_PREPARE(1, 8);
    else if (dtype == SCFA_BF16) SCFA_PREPARE(1, 16);
    else if (d == 64) SCFA_PREPARE(0, 8);
    else SCFA_PREPARE(0, 16);
#undef SCFA_PREPARE
    SCFA_HIP_TRY(hipGetLastError());
    return SCFA_OK;
}

// LDS of ranges_block: the searched vector is staged whole, or every 2^shift-th entry of it, within `most` bytes
static size_t ranges_smem(int T, int nb, int n_max, size_t most, int& shift)
{
    const size_t small = sizeof(int32_t) * ((4 * (size_t)(nb + 1) + (size_t)n_max + 3) & ~(size_t)3);
    shift = 0;
    while (small + sizeof(int32_t) * ((((size_t)T - 1) >> shift) + 1) > most && (T - 1) >> shift > 0) ++shift;
    return small + sizeof(int32_t) * ((((size_t)T - 1) >> shift) + 1);
}

int launch_block_ranges(int variant, const int32_t* q_idx, const int32_t* k_idx,
                        const int32_t* q_off, const int32_t* k_off, int S, int T, int nb,
                        int fwd_m, int fwd_n, int bwd_n, int bwd_m, int n_fwd, int n_bwd, int strict,
                        int32_t* fwd_work, int32_t* bwd_work, int64_t* counters, hipStream_t st)
{
    int shift;
    const size_t smem = ranges_smem(T, nb, n_fwd > n_bwd ? n_fwd : n_bwd, 144 * 1024, shift);
    static std::atomic<unsigned long long> lds_allowed{0};
    { const int rc_ = allow_dynamic_lds(reinterpret_cast<const void*>(&block_ranges_kernel), 144 * 1024, lds_allowed); if (rc_ != SCFA_OK) return rc_; }
    const RangesArgs ar{variant, q_idx, k_idx, q_off, k_off, T, nb, fwd_m, fwd_n, bwd_n, bwd_m, n_fwd, n_bwd, shift, strict,
                        fwd_work, bwd_work, (long long*)counters};
    ProfScope prof(SCFA_K_RANGES, st);
    hipLaunchKernelGGL(block_ranges_kernel, dim3(S, bwd_work ? 2 : 1), dim3(RANGES_THREADS), smem, st, ar);
    SCFA_HIP_TRY(hipGetLastError());
    return SCFA_OK;
}

// mode as in convert_chunk; q null: only K and V are gathered; the index vectors (positions or sort keys) serve both parts
int launch_gather_and_ranges(int variant, const void* q, const void* k, const void* v, void* q_p, void* k_p, void* v_p, int mode,
                             int d, const int32_t* q_idx, const int32_t* k_idx, const int32_t* q_off, const int32_t* k_off, int S,
                             int T, int nb, int n_fwd, int n_bwd, int strict, int32_t* fwd_work, int32_t* bwd_work,
                             int64_t* counters, hipStream_t st)
{
    // Staging at most 36 KiB keeps four 512-thread workgroups on a CU (the gather's occupancy); longer vectors are searched
    // through samples, a few dependent reads more beside a gather that takes longer than that.
    int shift;
    const int n_max = n_fwd > n_bwd ? n_fwd : n_bwd;
    const size_t smem = ranges_smem(T, nb, n_max, 36 * 1024 + 4 * (size_t)n_max, shift);
    const RangesArgs ar{variant, q_idx, k_idx, q_off, k_off, T, nb, FWD_TILE_M, FWD_TILE_N, BWD_TILE_N, BWD_TILE_M, n_fwd, n_bwd,
                        shift, strict, fwd_work, bwd_work, (long long*)counters};
    const bool drop = variant == SCFA_QKDROP;
    const GatherBatch batch{{{k, k_idx, drop ? k_off : nullptr, k_p, 1.f}, {v, k_idx, drop ? k_off : nullptr, v_p, 1.f},
                             {q, q_idx, drop ? q_off : nullptr, q_p, 1.f}}};
    const int n_tensors = q ? 3 : 2;
    const int cpr = d * 2 / 16, n_lists = S * (bwd_work ? 2 : 1);
    const int per_wg = RANGES_THREADS * GATHER_PER_THREAD;
    const long long per_seg = ((long long)T * cpr + per_wg - 1) / per_wg;
    const dim3 grid((unsigned)(n_lists + n_tensors * S * per_seg)), block(RANGES_THREADS);
    ProfScope prof(SCFA_K_GATHER, st);
    const auto launch = [&](auto kernel, std::atomic<unsigned long long>& lds_allowed) -> int {
        const int rc = allow_dynamic_lds(reinterpret_cast<const void*>(kernel), 144 * 1024, lds_allowed);
        if (rc != SCFA_OK) return rc;
        hipLaunchKernelGGL(kernel, grid, block, smem, st, ar, batch, S, n_lists, (int)per_seg, cpr);
        return SCFA_OK;
    };
    static std::atomic<unsigned long long> lds_allowed[4];   // one for each instantiation
    const bool stream = gather_streams(S, T, d * 2, bwd_work != nullptr, drop);
    const int rc = mode == 1 ? (stream ? launch(&gather_and_ranges_kernel<1, true>, lds_allowed[0]) : launch(&gather_and_ranges_kernel<1, false>, lds_allowed[1]))
                             : (stream ? launch(&gather_and_ranges_kernel<0, true>, lds_allowed[2]) : launch(&gather_and_ranges_kernel<0, false>, lds_allowed[3]));
    if (rc != SCFA_OK) return rc;
    SCFA_HIP_TRY(hipGetLastError());
    return SCFA_OK;
}

}  // namespace scfa
