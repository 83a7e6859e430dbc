// Keys, and the row gather, shared by the single entry points and by the launches that do several passes at once.  Gather:
// 16 bytes per thread, a row of d elements is row_bytes / 16 consecutive lanes, so every row is read and written as
// whole cache lines.
#pragma once

#include "scfa_common.hpp"

#include <type_traits>

namespace scfa {

// the key token i is sorted by: its bucket id, brought into [0, nb), or (KEEP_MODE: uint8 flags) 0 = kept, 1 = dropped
template <bool KEEP_MODE>
__device__ __forceinline__ int load_key(const void* keys, size_t i, int nb)
{
    if (KEEP_MODE) {
        return reinterpret_cast<const uint8_t*>(keys)[i] != 0 ? 0 : 1;
    } else {
        int k = reinterpret_cast<const int32_t*>(keys)[i];
        k = k < 0 ? 0 : k;
        return k >= nb ? nb - 1 : k;
    }
}

// sum over lanes 0 .. own of the wavefront
__device__ __forceinline__ int wave_prefix(int x)
{
    x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);   // row_shr:1, rows of 16 lanes
    x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);   // row_bcast:15 into rows 1 and 3
    x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);   // row_bcast:31 into rows 2 and 3
    return x;
}

// sum over the wavefront
__device__ __forceinline__ long long wave_total(long long x)
{
    auto step = [&](auto ctrl, auto rows) __attribute__((always_inline)) {
        const uint32_t lo = __builtin_amdgcn_update_dpp(0, (int)x, decltype(ctrl)::value, decltype(rows)::value, 0xf, false);
        const uint32_t hi = __builtin_amdgcn_update_dpp(0, (int)(x >> 32), decltype(ctrl)::value, decltype(rows)::value, 0xf, false);
        x += (long long)((unsigned long long)hi << 32 | lo);
    };
    step(std::integral_constant<int, 0x111>{}, std::integral_constant<int, 0xf>{});      // as in wave_prefix
    step(std::integral_constant<int, 0x112>{}, std::integral_constant<int, 0xf>{});
    step(std::integral_constant<int, 0x114>{}, std::integral_constant<int, 0xf>{});
    step(std::integral_constant<int, 0x118>{}, std::integral_constant<int, 0xf>{});
    step(std::integral_constant<int, 0x142>{}, std::integral_constant<int, 0xa>{});
    step(std::integral_constant<int, 0x143>{}, std::integral_constant<int, 0xc>{});
    const uint32_t lo = __builtin_amdgcn_readlane((int)x, 63), hi = __builtin_amdgcn_readlane((int)(x >> 32), 63);
    return (long long)((unsigned long long)hi << 32 | lo);
}

// Counts to places, by one wavefront, a key per lane: hist[w][k], the tokens of key k in the w-th of WAVES runs, becomes the place of
// the first of them, and off[k] that of the segment's first (off[nb]: all tokens).  others(k, earlier, later): tokens of the key in
// front of these runs and behind them.
template <int WAVES, typename F>
__device__ __forceinline__ void place_keys(int32_t* hist, int32_t* off, int nb, int lane, F others)
{
    int carry = 0;
    for (int b0 = 0; b0 < nb; b0 += 64) {
        const int k = b0 + lane;
        int c[WAVES], sum = 0, earlier = 0, later = 0;
        if (k < nb) {
#pragma unroll
            for (int w = 0; w < WAVES; ++w) c[w] = hist[w * nb + k];
            others(k, earlier, later);
#pragma unroll
            for (int w = 0; w < WAVES; ++w) sum += c[w];
            sum += earlier + later;
        }
        const int end = wave_prefix(sum) + carry;
        if (k < nb) {
            int at = end - sum;
            off[k] = at;
            at += earlier;
#pragma unroll
            for (int w = 0; w < WAVES; ++w) {
                hist[w * nb + k] = at;
                at += c[w];
            }
        }
        carry = __builtin_amdgcn_readlane(end, 63);
    }
    if (lane == 0) off[nb] = carry;
}

// lanes with this lane's key (of `nbits` bits) among those of `valid`
__device__ __forceinline__ unsigned long long same_key(int key, int nbits, unsigned long long valid)
{
    uint32_t lo = (uint32_t)valid, hi = (uint32_t)(valid >> 32);
    for (int b = 0; b < nbits; ++b) {
        const uint32_t other = ((uint32_t)key >> b & 1u) - 1u;       // all ones where the bit is 0
        const unsigned long long m = __ballot(other == 0);
        lo &= (uint32_t)m ^ other;
        hi &= (uint32_t)(m >> 32) ^ other;
    }
    return (unsigned long long)hi << 32 | lo;
}

struct GatherProblem {
    const void* x;
    const int32_t* idx;      // positions, or sort keys (their low bits are the positions)
    const int32_t* count;
    void* out;
    float scale;
};
struct GatherBatch { GatherProblem p[3]; };

// MODE 0: bit-exact copy; 1: bf16 -> fp16 (times scale, one rounding to nearest even; with
// scale 1 exact for magnitudes in [2^-17, 65504], larger ones become infinite and NaN stays
// NaN, so that an input outside the compute format shows in the results instead of being
// replaced by a finite value); 2: fp32 times scale (one rounding)
template <int MODE>
__device__ __forceinline__ uint4 convert_chunk(uint4 v, float scale)
{
    if (MODE == 1) {
        const uint32_t w[4] = {v.x, v.y, v.z, v.w};
        uint32_t o[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float lo = __uint_as_float(w[i] << 16) * scale, hi = __uint_as_float(w[i] & 0xffff0000u) * scale;
            const _Float16 a = (_Float16)lo, b = (_Float16)hi;   // IEEE conversion: beyond the fp16 range -> inf, NaN stays NaN
            o[i] = (uint32_t)__builtin_bit_cast(uint16_t, a) | ((uint32_t)__builtin_bit_cast(uint16_t, b) << 16);
        }
        return make_uint4(o[0], o[1], o[2], o[3]);
    } else if (MODE == 2) {
        return make_uint4(__float_as_uint(__uint_as_float(v.x) * scale), __float_as_uint(__uint_as_float(v.y) * scale),
                          __float_as_uint(__uint_as_float(v.z) * scale), __float_as_uint(__uint_as_float(v.w) * scale));
    }
    return v;
}

// Whether the rows of a gather are read past the caches.  Nobody reads them again, and where K and V do not fit the L2s together (32 MB;
// with a backward, where Q is copied as well, 22 MB) they would push out the copies that the attention reads.  Below, a caller's rows are
// often in the caches and come faster from there.  In us, through the caches / past them, inputs that were read a call ago (in brackets: that were
// written just before, with those writes); segments of 8192 rows where nothing else is said.
// Forward only, d = 64, 8 segments 38.6 / 40.3 (47.8 / 48.0), 12 42.3 / 46.3 (56.4 / 56.8), 16 49.3 / 51.9 (67.5 / 68.0), 20 56.8 / 60.0 (83.5 / 79.5),
// 32 80.4 / 79.5 (120.7 / 118.9), 48 111.6 / 106.8 (171.4 / 167.4); d = 128, 4 42.8 / 46.8 (51.6 / 52.0), 8 50.4 / 53.1 (67.9 / 68.2), 10 58.4 / 61.8
// (84.7 / 81.8).  Training step, 12 x 4164 65.7 / 68.9 (74.9 / 74.8), 8 83.2 / 84.7 (94.6 / 94.7), 10 95.4 / 97.3 (108.1 / 109.4), 12 105.2 / 108.1 (123.0 /
// 121.2), 16 127.7 / 130.7 (152.4 / 150.8), 24 181.4 / 176.0 (210.6 / 210.1), 96 x 4096 296.8 / 287.8 (359.8 / 349.5).
// QK-dropping reads the rows it keeps, taken as half of them.  Half kept, forward, 16 x 8192 x 128 120.9 / 124.8 (163.1 / 162.5), 16 x 16384 200.2 / 203.6
// (243.7 / 242.3), 24 x 16384 278.8 / 278.8 (337.5 / 336.8); training step, 16 224.0 / 227.7 (247.2 / 246.0), 20 262.2 / 265.8 (290.8 / 290.7).
inline bool gather_streams(long long S, long long T, int row_bytes, bool train, bool drop)
{
    return S * T * row_bytes > (train ? 11LL : 16LL) * (drop ? 2 : 1) << 20;
}

// chunks g0 + i * stride (i < N) of segment s: the N index reads, then the N row reads of a thread are in flight together.  (STREAM as an
// argument and both forms of the reads in the kernel: 192 x 1024 rows 54.3 -> 57.1 us.)
template <int MODE, int N, bool STREAM>
__device__ __forceinline__ void gather_chunks(const GatherProblem& pr, int s, long long g0, int stride, int T, int chunks_per_row,
                                              int32_t pos_mask)
{
    const int n = pr.count ? pr.count[s] : T;
    const int32_t* __restrict__ idx = pr.idx + (size_t)s * T;
    const uint4* __restrict__ x = reinterpret_cast<const uint4*>(pr.x) + (size_t)s * T * chunks_per_row;
    uint4* __restrict__ out = reinterpret_cast<uint4*>(pr.out) + (size_t)s * T * chunks_per_row;
    int r[N], src[N];
    uint4 v[N];
#pragma unroll
    for (int i = 0; i < N; ++i) {
        r[i] = (int)((g0 + (long long)i * stride) / chunks_per_row);
        src[i] = r[i] < n ? idx[r[i]] & pos_mask : 0;
    }
    const int c = (int)(g0 % chunks_per_row);        // the stride is a whole number of rows
#pragma unroll
    for (int i = 0; i < N; ++i)
        if (r[i] < n) {
            const uint4* const from = x + (size_t)src[i] * chunks_per_row + c;
            v[i] = STREAM ? load_stream(from) : *from;
        }
#pragma unroll
    for (int i = 0; i < N; ++i)
        if (r[i] < n) out[(size_t)r[i] * chunks_per_row + c] = convert_chunk<MODE>(v[i], pr.scale);
}

}  // namespace scfa
