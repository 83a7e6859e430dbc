// Shared declarations of the HIP sources of the SCFA library (gfx950 only).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>
#include <atomic>

#include "scfa.h"

namespace scfa {

// ---- error plumbing ---------------------------------------------------------
extern thread_local int g_last_hip_error;

inline int hip_fail(hipError_t e)
{
    g_last_hip_error = (int)e;
    return SCFA_EHIP;
}

#define SCFA_HIP_TRY(expr)                                 \
    do {                                                   \
        hipError_t _e = (expr);                            \
        if (_e != hipSuccess) return ::scfa::hip_fail(_e); \
    } while (0)

// A kernel that takes more than 64 KB of dynamic LDS has to be told so once on every device it
// runs on.  `done` (one per kernel instantiation) remembers the devices already prepared, one
// bit each; the current device is the one the caller's stream belongs to.
inline int allow_dynamic_lds(const void* kernel, int bytes, std::atomic<unsigned long long>& done)
{
    int dev = 0;
    SCFA_HIP_TRY(hipGetDevice(&dev));
    const unsigned long long bit = 1ull << (dev & 63);
    if (done.load(std::memory_order_acquire) & bit) return SCFA_OK;
    SCFA_HIP_TRY(hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes));
    done.fetch_or(bit, std::memory_order_release);
    return SCFA_OK;
}

// ---- profiling hooks (scfa_prof_*) -----------------------------------------
struct ProfScope {
    int kid;
    hipStream_t stream;
    int slot;
    ProfScope(int kernel_id, hipStream_t s);
    ~ProfScope();
};
bool prof_enabled();

// ---- work list layout (see scfa_block_ranges) -------------------------------
constexpr int WORK_STRIDE = SCFA_WORK_STRIDE;

// forward / dQ items
constexpr int W_QBEGIN = 0, W_QCOUNT = 1, W_KBEGIN = 2, W_KCOUNT = 3, W_KNOMASK = 4, W_BUCKET = 5, W_NBUCKETS = 6;
// backward (key-major) items
constexpr int BW_KBEGIN = 0, BW_KCOUNT = 1, BW_QBEGIN = 2, BW_QCOUNT = 3, BW_QMASKED = 4;

// ---- sort keys ------------------------------------------------------------------
// The attention kernels identify a sorted row by its sort key, bucket << 24 | original position
// (scfa_sort_by_bucket's sort_key_out; a compacted index vector of QK-dropping is its own key,
// the one bucket having id 0).  Keys increase along the sorted rows of a segment, and "same
// bucket, position <= p" is one unsigned range test: (key - (bucket << 24)) <= p.
constexpr uint32_t KEY_POS_BITS = 24;
constexpr uint32_t KEY_POS_MASK = (1u << KEY_POS_BITS) - 1u;
constexpr uint32_t KEY_PAST_END = 0xffffffffu;   // rows past the end of a ragged tile: match no range
constexpr uint32_t KEY_NEVER = 0xfffffffeu;      // lower end of the range of a row that may match nothing

// ---- streams ----------------------------------------------------------------------
// Sixteen bytes that no kernel of a forward or a training step reads again (a backward that is given no fp16 copy of O reads O).  As ordinary
// stores the results of a training step (O, the fp32 gradients,
// zeros of dropped rows: 350 MB at 48 x 8192 x 64 rows) take the place of the permuted copies in L2 and the 256 MB behind it, which
// the kernels still read: 373 -> 355 us a step there, 36 x 5003 rows 184 -> 176, 192 x 1024 169 -> 161, 24 x 16384 698 -> 678.  Only for
// instructions that write whole cache lines: smaller pieces are then not put together any more (dK/dV with 32-byte pieces 40 % slower
// at 24 x 16384 rows, 2.5 times at 48 x 8192).
// Whoever reads the results next finds less of them in the caches.  With O transposed and the gradients rounded to bf16 right behind the
// step, ordinary / streaming stores, without these readers in brackets: 32 x 1024 rows 71.6 / 72.0 (47.8 / 45.7), 32 x 2048 92.4 / 92.6 (67.8 / 65.7),
// 16 x 8192 177.9 / 177.8 (135.2 / 129.8), 192 x 1024 232.3 / 228.7 (168.4 / 160.2), 32 x 8192 329.9 / 318.8 (246.8 / 231.8), 48 x 8192 471.8 /
// 465.2 (356.5 / 338.7), 32 x 4096 x 128 341.1 / 324.1 (253.7 / 240.3), QK-dropping 16 x 4096 x 128 161.4 / 163.6 (118.4 / 114.2): up to about
// 130000 rows of 64 the reader loses what the step gains, above both gain.
typedef unsigned int u32v4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ void store_stream(uint4* p, uint4 x) { __builtin_nontemporal_store(__builtin_bit_cast(u32v4, x), reinterpret_cast<u32v4*>(p)); }
__device__ __forceinline__ uint4 load_stream(const uint4* p) { return __builtin_bit_cast(uint4, __builtin_nontemporal_load(reinterpret_cast<const u32v4*>(p))); }

// ---- tile configuration -------------------------------------------------------
constexpr int FWD_TILE_M = 128;  // query rows per workgroup (4 waves x 32)
constexpr int FWD_TILE_N = 64;   // keys per inner step
constexpr int BWD_TILE_N = 128;  // key rows per workgroup in the dK/dV kernel (4 waves x 32)
constexpr int BWD_TILE_M = 64;   // query rows per inner step of the dK/dV kernel
constexpr int F32_TILE_M = 64;   // fp32 path: query rows per workgroup (2 waves x 32, times the key splits)
constexpr int F32_TILE_N = 32;   // keys per tile of one wave

// ---- which segment and work rank a workgroup takes ---------------------------------------------
// Workgroup b of a launch of the fp16 attention kernels takes work rank b / S of a segment: the longest items of every segment are dispatched first.
// Workgroups go round the 8 XCDs, and the ranks are turned by (b / S) S mod 8 places so that a segment meets the same XCD, and its
// streams that XCD's L2, at every rank, but for the up to 7 segments at the turn.  (Not up to 8 segments, most of which would be at
// the turn.)  Training step in us, as they come / turned: 30 x 1500 rows 58.5 / 56.0, 100 x 2000 174.2 / 169.6, 36 x 5003 172.9 / 170.8,
// 18 x 3500 x 128 147.8 / 145.0, 20 x 8192 147.0 / 144.6, 36 x 8192 261.9 / 261.1; QK-dropping 20 x 1000 51.4 / 49.4, 9 x 20000 551 / 543.
// (fp32, whose rows are read in place: 30 x 1000 33.2 / 32.9, but 20 x 2000 x 128 97.2 / 98.6: left as they come.)
__device__ __forceinline__ void place_workgroup(int b, int S, int& s, int& rank)
{
    rank = b / S;
    s = b - rank * S;
    if (S > 8) {
        s += (b - s) & 7;
        if (s >= S) s -= S;
    }
}

// ---- grids beyond 2^32 threads ---------------------------------------------------------------
// A launch whose threads do not fit 32 bits runs only part of its workgroups and reports no error.  The attention kernels take a
// workgroup per work item and segment, item-major, and the items from `first` on: launch(first, items) is called for as many
// items at a time as one grid takes (all of them but with tens of thousands of segments and hundreds of items each).
template <typename F>
int launch_in_grids(int S, long long items, int threads, F launch)
{
    const long long most = 0xffffffffLL / ((long long)S * threads);     // S <= 65535, threads <= 512: at least 128
    for (long long first = 0; first < items; first += most) {
        const int rc = launch((int)first, (unsigned)(items - first < most ? items - first : most));
        if (rc != SCFA_OK) return rc;
    }
    return SCFA_OK;
}

// ---- kernel launchers (defined in the .hip files) ---------------------------
int launch_sort_by_bucket(int n_problems, const int32_t* bucket0, const int32_t* bucket1, int S, int T, int nb,
                          int32_t* idx0, int32_t* sorted0, int32_t* off0, uint32_t* key0, int32_t* idx1,
                          int32_t* sorted1, int32_t* off1, uint32_t* key1, void* ws, size_t ws_bytes, hipStream_t st);
int launch_count_invalid_buckets(const int32_t* bucket, long long n, int nb, int32_t* counter, hipStream_t st);
int launch_sort_by_bucket_static(const int32_t* bucket, int S, int T, int nb, int32_t* idx, int32_t* sorted,
                                 int32_t* off, uint32_t* key, hipStream_t st);
int launch_compact_keep(int n_problems, const uint8_t* keep0, const uint8_t* keep1, int S, int T, int32_t* idx0,
                        int32_t* count0, int32_t* idx1, int32_t* count1, void* ws, size_t ws_bytes, hipStream_t st);
size_t sort_workspace_bytes(int n_problems, int S, int T, int nb);
int launch_lsh_buckets(int n_problems, const void* x0, const void* x1, const float* R, int S, int H, int T, int d,
                       int nb, bool bf16, int32_t* out0, int32_t* out1, hipStream_t st);
int launch_gather_rows(int n_tensors, const void* const* x, const int32_t* const* idx, const int32_t* const* count,
                       const float* scale, void* const* out, int S, int T, int row_bytes, int mode, hipStream_t st);
int launch_block_ranges(int variant, const int32_t* q_idx, const int32_t* k_idx,
                        const int32_t* q_off, const int32_t* k_off, int S, int T, int nb,
                        int fwd_m, int fwd_n, int bwd_n, int bwd_m, int n_fwd, int n_bwd, int strict,
                        int32_t* fwd_work, int32_t* bwd_work, int64_t* counters, hipStream_t st);
int launch_gather_and_ranges(int variant, const void* q, const void* k, const void* v, void* q_p, void* k_p, void* v_p, int mode,
                             int d, const int32_t* q_idx, const int32_t* k_idx, const int32_t* q_off, const int32_t* k_off, int S,
                             int T, int nb, int n_fwd, int n_bwd, int strict, int32_t* fwd_work, int32_t* bwd_work,
                             int64_t* counters, hipStream_t st);
bool prepare_in_one(int S, int T);   // sort, lists and gather in one launch
int launch_prepare(int variant, const void* label_q, const void* label_k, const void* q, const void* k, const void* v, void* q_p,
                   void* k_p, void* v_p, int dtype, int d, int S, int T, int nb, int n_fwd, int n_bwd, int strict, uint32_t* q_key,
                   uint32_t* k_key, int32_t* q_off, int32_t* k_off, int32_t* fwd_work, int32_t* bwd_work, int64_t* counters, hipStream_t st);
bool f32_in_one(int variant, int S, int T, int d, int nb, int n_work);   // fp32 forward: sort, list and attention in one launch
int launch_f32_one(int variant, const float* q, const float* k, const float* v, const void* label_q, const void* label_k, int S, int T,
                   int d, int nb, int n_work, float tau, int strict, uint32_t* q_key, uint32_t* k_key, int32_t* q_off, int32_t* k_off,
                   int32_t* work, int64_t* counters, float* o, float* lse, hipStream_t st);
int launch_attn_fwd_f32(const float* q, const float* k, const float* v, const uint32_t* q_key,
                        const uint32_t* k_key, const int32_t* work, int n_work, int S, int T, int d,
                        float tau, int strict, float* o, float* lse, const int32_t* n_keep_q, bool indirect,
                        hipStream_t st);   // n_keep_q as below; indirect: q, k, v in original order
int launch_attn_fwd_bf16(const void* q, const void* k, const void* v, const uint32_t* q_key,
                         const uint32_t* k_key, const int32_t* work, int n_work, int S, int T, int d,
                         float tau, int strict, void* o, float* lse, void* o_f16, const int32_t* n_keep_q, bool own_q, void* q_out,
                         hipStream_t st);   // own_q: q in original order, its permuted copy goes to q_out (nullable); n_keep_q: QK-dropping (the kernel writes the dropped rows), else null
size_t bwd_row_stats_bytes(int S, int T);
int launch_bwd_prep_bf16(const void* o, const void* o_f16, const float* lse, const void* d_o, const uint32_t* q_key,
                         const int32_t* n_q, int S, int T, int d, float tau, void* do_perm, void* row_perm,
                         void* aux_perm, void* row_stats, hipStream_t st);
int launch_attn_bwd_bf16(const void* q, const void* k, const void* v, const void* d_o, const void* do_perm, const void* aux_perm,
                         const void* row_perm, const void* row_stats, const uint32_t* q_key,
                         const uint32_t* k_key, const int32_t* fwd_work, int n_fwd, const int32_t* bwd_work, int n_bwd, int S, int T,
                         int d, float tau, int strict, float* dq, float* dk, float* dv, const int32_t* n_keep_q,
                         const int32_t* n_keep_k, hipStream_t st);   // n_keep_*: QK-dropping (the kernels zero the dropped rows), else null

int occupancy_attn_fwd_bf16(int d, int* out);
int occupancy_attn_bwd_dkdv_bf16(int d, int* out);
int occupancy_attn_bwd_dq_bf16(int d, int* out);

}  // namespace scfa
