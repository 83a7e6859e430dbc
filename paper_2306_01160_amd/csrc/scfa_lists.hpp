// The sort of a segment inside one workgroup, and the building of a work list, for the launches that do them beside or in front
// of something else.
#pragma once

#include "scfa_common.hpp"
#include "scfa_rows.hpp"

namespace scfa {

// The index vectors are positions or sort keys (bucket << 24 | position): the position is the low bits of both.
__device__ __forceinline__ int position(int32_t x) { return x & (int32_t)KEY_POS_MASK; }

// number of entries of a[0..n) with a position < v (positions increase along a)
__device__ __forceinline__ int count_below(const int32_t* __restrict__ a, int n, int v)
{
    int lo = 0, hi = n;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (position(a[mid]) < v) lo = mid + 1; else hi = mid;
    }
    return lo;
}

// The searched vector: `g` in global memory and lds[i] = g[i << shift] (shift 0: all of it).
struct Searched { const int32_t* g; const int32_t* lds; int shift; };

// number of entries of g[begin, begin + n) with a position < v, from samples
__device__ __forceinline__ int count_sampled(const Searched& a, int begin, int n, int v)
{
    int lo = begin, hi = begin + n;                        // the answer is a position in [lo, hi]
    const int j0 = (begin + (1 << a.shift) - 1) >> a.shift, j1 = (begin + n - 1) >> a.shift;   // samples inside
    if (n > 0 && j0 <= j1) {
        const int c = count_below(a.lds + j0, j1 - j0 + 1, v);
        if (c > 0) lo = ((j0 + c - 1) << a.shift) + 1;     // that sample and all before it count
        if (c <= j1 - j0) hi = (j0 + c) << a.shift;        // the next sample does not
    }
    return lo - begin + count_below(a.g + lo, hi - lo, v);
}

// ... for two values, the dependent reads of the two searches in flight together
__device__ __forceinline__ void count_below2(const Searched& a, int begin, int n, int v0, int v1, int& c0, int& c1)
{
    if (a.shift != 0) {
        c0 = count_sampled(a, begin, n, v0);
        c1 = count_sampled(a, begin, n, v1);
        return;
    }
    const int32_t* p = a.lds + begin;
    int lo0 = 0, hi0 = n, lo1 = 0, hi1 = n;
    while (lo0 < hi0 || lo1 < hi1) {
        const int m0 = (lo0 + hi0) >> 1, m1 = (lo1 + hi1) >> 1;
        const int x0 = position(p[min(m0, n - 1)]), x1 = position(p[min(m1, n - 1)]);
        if (lo0 < hi0) { if (x0 < v0) lo0 = m0 + 1; else hi0 = m0; }
        if (lo1 < hi1) { if (x1 < v1) lo1 = m1 + 1; else hi1 = m1; }
    }
    c0 = lo0;
    c1 = lo1;
}

constexpr int ORDER_GROUP = 2;   // buckets whose items are dispatched together

struct Item { int a_begin, a_count, b_begin, b_count, b_extra, unit; };

// ascending sort key: bucket pair first, then decreasing length of the ranged side (< 2^24)
__device__ __forceinline__ int order_key(int bucket, int b_count)
{
    return ((bucket / ORDER_GROUP) << 24) | (0xffffff - min(b_count, 0xffffff));
}

// Builds one work list.  Latency-bound: a few dependent LDS reads per phase, and the instructions themselves, which come from L2 the
// first time (one body for both lists and both mask forms: with one each, four in a kernel, the gather in the same launch took 42 us
// instead of 39 at 32 x 7001 x 128).  The two searches of an item run together and the items of its bucket pair are read off its unit's
// neighbours; with one search after the other and the pair found by search the launch took 12.1 us instead of 9.4 for 32 x 2048
// rows in fp32, and 1 x 256 rows 17.1 us a call instead of 16.0.  "a" is the tiled side (queries forward, keys backward),
// "b" the ranged side.
//   forward : b range = keys with pos <= max a pos;  extra = #keys with pos <= min a pos
//   backward: b range = queries with pos >= min a pos; extra = #queries of the range with pos < max a pos
// strict (a key is visible only to later positions, App. B.1's ">" in place of ">="): the
// comparisons with equality swap sides, <= becomes < and >= becomes >.
template <int THREADS>
__device__ __forceinline__ void build_list(bool forward, int strict, const int32_t* __restrict__ a_idx, const Searched& b_idx,
                           const int32_t* a_off, const int32_t* b_off, int nb, int tile_a,
                           int tile_b, int n_items_max, int32_t* __restrict__ work_out,
                           long long* counters2, int32_t* s_tile_base, int32_t* s_unit_first, int32_t* s_cost)
{
    // Units (nb <= 256): a bucket with a tile or more of rows on either side is a
    // unit of its own (its items keep their causal range and mask-free prefix); consecutive buckets
    // that are shorter than a tile on both sides are taken together while their rows on the tiled
    // side fit one tile: only there does one item walk fewer tiles than one item per bucket would.
    // Buckets of up to two tiles on the ranged side stay apart although sharing items is faster (training step of 192 x 1024 rows in
    // 16 buckets 158 -> 151 us): masked values are multiplied by 0, so a value that is not finite would reach the rows of the
    // buckets beside its own, and dK / dV would be formed on the scale of the largest dO of them all.
    // Tiles per unit -> exclusive prefix.  The merge is a serial scan over the buckets; one wavefront holds the bucket
    // sizes in its lanes and reads them out as scalars (a scan over LDS by one thread cost its LDS latency three times per
    // bucket: 16 us of schedule at 32 buckets, 72 segments).
    __shared__ int s_n_units;
    if (threadIdx.x < 64) {
        // the rows of lane b's bucket
        const int lane = threadIdx.x, mine = min(lane, nb - 1);
        const int ra0 = a_off[mine + 1] - a_off[mine], rb0 = b_off[mine + 1] - b_off[mine];
        if (nb <= 64) {
            // whether the next bucket could join lane b's; often no neighbours are so short
            const int after = min(lane + 1, nb - 1), ra1 = a_off[after + 1] - a_off[after], rb1 = b_off[after + 1] - b_off[after];
            if (__ballot(lane < nb - 1 && ra0 < tile_a && max(rb0, rb1) < tile_b && ra0 + ra1 <= tile_a) == 0) {
                const int n = lane < nb ? (ra0 + tile_a - 1) / tile_a : 0, end = wave_prefix(n);
                if (lane < nb) { s_unit_first[lane] = lane; s_tile_base[lane] = end - n; }
                if (lane == nb - 1) { s_unit_first[nb] = nb; s_tile_base[nb] = end; s_n_units = nb; }
            } else {
                unsigned long long firsts = 0;     // bit b: bucket b is the first of a unit
                int rows = 0;
                bool open = false;                 // the unit being built may take further buckets
                for (int b = 0; b < nb; ++b) {
                    const int ra = __builtin_amdgcn_readlane(ra0, b), rb = __builtin_amdgcn_readlane(rb0, b);
                    if (open && rb < tile_b && rows + ra <= tile_a) {
                        rows += ra;
                    } else {
                        firsts |= 1ull << b;
                        rows = ra;
                        open = ra < tile_a && rb < tile_b;
                    }
                }
                const unsigned long long here = 1ull << lane, behind = firsts & ~(here | (here - 1));
                const bool first = (firsts & here) != 0;
                const int n = first ? (a_off[behind ? __builtin_ctzll(behind) : nb] - a_off[lane] + tile_a - 1) / tile_a : 0, end = wave_prefix(n);
                const int u = __popcll(firsts & (here - 1)), n_units = __popcll(firsts);
                if (first) { s_unit_first[u] = lane; s_tile_base[u] = end - n; }
                if (lane == nb - 1) { s_unit_first[n_units] = nb; s_tile_base[n_units] = end; s_n_units = n_units; }
            }
        } else {
            int acc = 0, u = 0, rows = 0;
            bool open = false;     // the unit being built may take further buckets
            for (int b0 = 0; b0 < nb; b0 += 64) {
                const int mine = min(b0 + (int)threadIdx.x, nb - 1);
                const int ra_lane = a_off[mine + 1] - a_off[mine], rb_lane = b_off[mine + 1] - b_off[mine];
                const int n = min(64, nb - b0);
                for (int i = 0; i < n; ++i) {
                    const int ra = __builtin_amdgcn_readlane(ra_lane, i), rb = __builtin_amdgcn_readlane(rb_lane, i);
                    if (open && rb < tile_b && rows + ra <= tile_a) {
                        rows += ra;
                        continue;
                    }
                    acc += (rows + tile_a - 1) / tile_a;         // the unit before is complete
                    if (threadIdx.x == 0) { s_unit_first[u] = b0 + i; s_tile_base[u] = acc; }
                    ++u;
                    rows = ra;
                    open = ra < tile_a && rb < tile_b;
                }
            }
            acc += (rows + tile_a - 1) / tile_a;
            if (threadIdx.x == 0) { s_unit_first[u] = nb; s_tile_base[u] = acc; s_n_units = u; }
        }
    }
    __syncthreads();
    const int n_units = s_n_units;
    const int n_items = s_tile_base[n_units];

    auto make_item = [&](int w) -> Item {
        // unit of item w: last u with tile_base[u] <= w
        int lo = 0, hi = n_units - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (s_tile_base[mid] <= w) lo = mid; else hi = mid - 1;
        }
        const int b = s_unit_first[lo];
        const int b_last = s_unit_first[lo + 1] - 1;
        Item it;
        it.unit = lo;
        if (b_last > b) {   // several small buckets: all their rows on both sides, every tile tested
            it.a_begin = a_off[b];
            it.a_count = a_off[b_last + 1] - a_off[b];
            it.b_begin = b_off[b];
            it.b_count = b_off[b_last + 1] - b_off[b];
            it.b_extra = forward ? 0 : it.b_count;
            return it;
        }
        it.a_begin = a_off[b] + (w - s_tile_base[lo]) * tile_a;
        it.a_count = min(tile_a, a_off[b + 1] - it.a_begin);
        const int pos_min = position(a_idx[it.a_begin]);
        const int pos_max = position(a_idx[it.a_begin + it.a_count - 1]);
        const int bb = b_off[b], bn = b_off[b + 1] - b_off[b];
        // the ranged rows in front of the tile's first and of its last row: keys at its position too, unless strict; queries at its
        // position only if strict
        const int shift = forward ? 1 - strict : strict;
        int first, last;
        count_below2(b_idx, bb, bn, pos_min + shift, pos_max + shift, first, last);
        it.b_begin = forward ? bb : bb + first;
        it.b_count = forward ? last : bn - first;
        it.b_extra = forward ? first : max(last - first, 0);
        return it;
    };

    // the first KEEP items of a thread stay in registers between the two passes (their range
    // ends cost dependent memory reads); beyond that they are computed again
    constexpr int KEEP = 4;
    Item kept[KEEP];
    for (int w = threadIdx.x, j = 0; w < n_items; w += THREADS, ++j) {
        const Item it = make_item(w);
        s_cost[w] = order_key(s_unit_first[it.unit], it.b_count);
#pragma unroll
        for (int u = 0; u < KEEP; ++u) if (j == u) kept[u] = it;   // register selects, no indexing
    }
    __syncthreads();

    long long tiles = 0, rect = 0;
    for (int w = threadIdx.x, j = 0; w < n_items_max; w += THREADS, ++j) {
        if (w < n_items) {
            Item it;
            if (j < KEEP) {
                it = kept[0];
#pragma unroll
                for (int u = 1; u < KEEP; ++u) if (j == u) it = kept[u];
            } else {
                it = make_item(w);
            }
            const int bucket = s_unit_first[it.unit], c = order_key(bucket, it.b_count);
            // items are generated in unit order, so those of one bucket pair are a run [lo, hi) of w: the unit's and its neighbours'
            const int pair = c >> 24;
            int u0 = it.unit, u1 = it.unit + 1;
            while (u0 > 0 && s_unit_first[u0 - 1] / ORDER_GROUP == pair) --u0;
            while (u1 < n_units && s_unit_first[u1] / ORDER_GROUP == pair) ++u1;
            const int lo = s_tile_base[u0], hi = s_tile_base[u1];
            int rank = lo;
#pragma unroll 4
            for (int u = lo; u < hi; ++u) {
                const int cu = s_cost[u];
                rank += (cu < c) || (cu == c && u < w);
            }
            int32_t* o = work_out + (size_t)rank * WORK_STRIDE;
            o[0] = it.a_begin; o[1] = it.a_count; o[2] = it.b_begin; o[3] = it.b_count;
            o[4] = it.b_extra; o[5] = bucket; o[6] = s_unit_first[it.unit + 1] - bucket; o[7] = 0;
            tiles += (it.b_count + tile_b - 1) / tile_b;
            rect += (long long)it.a_count * it.b_count;
        } else {
            int32_t* o = work_out + (size_t)w * WORK_STRIDE;
#pragma unroll
            for (int i = 0; i < WORK_STRIDE; ++i) o[i] = 0;
        }
    }
    // block reduction of the two counters
    __shared__ long long s_red[2][THREADS / 64];
    tiles = wave_total(tiles);
    rect = wave_total(rect);
    if ((threadIdx.x & 63) == 0) { s_red[0][threadIdx.x >> 6] = tiles; s_red[1][threadIdx.x >> 6] = rect; }
    __syncthreads();
    if (threadIdx.x == 0 && counters2) {
        long long t = 0, r = 0;
        for (int i = 0; i < THREADS / 64; ++i) { t += s_red[0][i]; r += s_red[1][i]; }
        counters2[0] = t; counters2[1] = r;
    }
    __syncthreads();
}

// Stable sort of T <= 64 * STEPS * WAVES tokens by WAVES wavefronts, the scheme of scfa_index.hip in one workgroup; the other
// half of the workgroup runs the same steps (barriers) on the other side.  off[0 .. nb]: start of every key; sorted: sort keys
// (KEEP_MODE: positions).  hist: [WAVES][nb].
// With two keys 64 atomics on their counters are served nearly one after the other, and a ballot ranks a step: up to two keys (TWO)
// are ranked while they are counted (one bucket of 4096 rows, forward 58.4 -> 51.8 us; QK-dropping training step at 32 x 2048 rows
// 71.2 -> 69.3 us, this launch 12.9 -> 11.3).  With more keys the atomics are the cheaper count (hash forward in fp32, 256 rows in 4
// buckets: 17.8 -> 18.0 us ranked at once).
template <int WAVES, int STEPS, bool KEEP_MODE, bool TWO>
__device__ __forceinline__ void sort_side(const void* __restrict__ keys, size_t seg, int T, int nb, int nbits, int wave, int lane,
                                          int32_t* hist, int32_t* off, uint32_t* sorted)
{
    static_assert(TWO || !KEEP_MODE, "without TWO the sorted words are sort keys");
    const int ht = wave * 64 + lane;
    int run = (T + WAVES - 1) / WAVES;
    run = (run + 63) & ~63;
    const int r0 = min(wave * run, T), r1 = min(r0 + run, T);
    int keyv[STEPS];
#pragma unroll
    for (int u = 0; u < STEPS; ++u) {
        const int t = r0 + 64 * u + lane;
        keyv[u] = t < r1 ? load_key<KEEP_MODE>(keys, seg + t, nb) : -1;
    }
    for (int i = ht; i < WAVES * nb; i += 64 * WAVES) hist[i] = 0;
    __syncthreads();
    const unsigned long long lt_mask = (1ull << lane) - 1ull;
    int seen[2] = {0, 0};                                  // TWO: this wavefront's tokens of either key
    if constexpr (TWO) {
#pragma unroll
        for (int u = 0; u < STEPS; ++u) {
            const unsigned long long m0 = __ballot(keyv[u] == 0), m1 = __ballot(keyv[u] == 1);
            if (keyv[u] >= 0) keyv[u] |= (keyv[u] ? seen[1] + __popcll(m1 & lt_mask) : seen[0] + __popcll(m0 & lt_mask)) << 1;   // place, key
            seen[0] += __popcll(m0);
            seen[1] += __popcll(m1);
        }
        if (lane < min(nb, 2)) hist[wave * nb + lane] = lane ? seen[1] : seen[0];
    } else {
#pragma unroll
        for (int u = 0; u < STEPS; ++u)
            if (keyv[u] >= 0) atomicAdd(&hist[wave * nb + keyv[u]], 1);
    }
    __syncthreads();
    if (wave == 0) place_keys<WAVES>(hist, off, nb, lane, [](int, int&, int&) {});
    __syncthreads();
    int32_t* base = hist + wave * nb;
    if constexpr (TWO) {
        const int first[2] = {base[0], nb > 1 ? base[1] : 0};
#pragma unroll
        for (int u = 0; u < STEPS; ++u)
            if (keyv[u] >= 0)
                sorted[(keyv[u] & 1 ? first[1] : first[0]) + (keyv[u] >> 1)] =
                    (KEEP_MODE ? 0u : (uint32_t)(keyv[u] & 1) << KEY_POS_BITS) | (uint32_t)(r0 + 64 * u + lane);
        __syncthreads();
        return;
    }
#pragma unroll
    for (int u = 0; u < STEPS; ++u) {
        const int t = r0 + 64 * u + lane;
        if (r0 + 64 * u >= r1) break;                      // wave-uniform
        const bool valid = t < r1;
        const int key = valid ? keyv[u] : 0;
        const unsigned long long same = same_key(key, nbits, __ballot(valid));
        const int rank = __popcll(same & lt_mask);
        int at = 0, pos = 0;
        if (valid) { at = base[key]; pos = at + rank; }
        __builtin_amdgcn_wave_barrier();
        if (valid && rank == 0) base[key] = at + __popcll(same);
        __builtin_amdgcn_wave_barrier();
        if (valid) sorted[pos] = (uint32_t)key << KEY_POS_BITS | (uint32_t)t;
    }
    __syncthreads();
}

}  // namespace scfa
