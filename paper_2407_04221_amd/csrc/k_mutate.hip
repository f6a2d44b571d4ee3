// Batched mutation operators (paper Sec. 2.2.1 and the Fig. 2b caption): environments are
// mutated by flipping bits of their initial multi-hot maps, by changing entries of their
// rules' input and output patterns, and by redrawing rule rewards.  Every individual of a
// population is mutated independently; each thread owns one Philox block (eight 32-bit
// words) and the elements those words decide, so the kernels are embarrassingly parallel,
// read and write each element once, and may run in place.
//
// What bounds them is the generator: 80 multiply-adds of 32 x 32 + 64 bits per block.  So a
// block's elements are moved as one word (eight cells or four entries; byte by byte they cost
// as much again), an entry's place in its pattern is counted on from the block's first, and rule
// sets take one launch for entries and rewards.  Measured (MI355X, 4096 individuals, maps of
// 8 x 32 x 32, 16 rules of 9 x 3 x 3 entries): both calls in a row 92 -> 69 us; each waited for,
// the kernels take 36.5 (maps) and 41.3 (rules).
//
//   maps     element e = (c * H + y) * W + x of individual k: one word (stream 1, word e);
//            flip iff channel c is allowed and the word is below the flip threshold;
//   entries  element e = (((r * 2 + io) * (C+1) + c) * mh + i) * mw + j of set s: two words
//            (stream 2, words 2e and 2e + 1); inside the rule's n x m and on an allowed
//            channel, change iff word 2e is below the entry threshold, to the lower (word
//            2e + 1 even) or higher (odd) of the two other values of {-1, 0, 1};
//   rewards  rule r of set s: stream 3, words 2r (redraw iff below the reward threshold)
//            and 2r + 1 (new reward lo + word mod (hi - lo + 1)).
#include <algorithm>

#include "av_internal.h"
#include "philox.h"

namespace av {
namespace {

// One thread per Philox block (eight elements).  With kRow a grid row is an individual, so the
// counter words that name it are scalar and the first two rounds take 6 of their 16
// multiply-adds from the vector unit; else thread t covers block t % blocks_per of individual
// k0 + t / blocks_per (32-bit index arithmetic: the launcher splits populations into chunks
// that fit).  The eight bytes are handled as one 64-bit word at any alignment.
template <bool kRow>
__global__ void __launch_bounds__(256) mutate_maps_kernel(const uint8_t *src, uint8_t *dst,
                                                          int k0, int nk, int per, int plane,
                                                          int blocks_per, int all_channels,
                                                          MutateArgs m) {
    const uint32_t t = blockIdx.x * blockDim.x + threadIdx.x;
    uint32_t kk, blk;
    if (kRow) {
        kk = blockIdx.y;
        blk = t;
        if (blk >= uint32_t(blocks_per)) return;
    } else {
        if (t >= uint32_t(nk) * uint32_t(blocks_per)) return;
        kk = t / uint32_t(blocks_per);
        blk = t - kk * uint32_t(blocks_per);
    }
    const uint32_t k = uint32_t(k0) + kk;
    const int e0 = int(blk) * 8;
    const uint8_t *s = src + size_t(k) * per + e0;
    uint8_t *d = dst + size_t(k) * per + e0;
    const bool whole = e0 + 8 <= per;
    uint64_t v = 0;
    if (whole) __builtin_memcpy(&v, s, 8);
    uint32_t w[8];
    philox_words(m.seed, m.generation, k, 1, blk, w);
    uint32_t lo = 0, hi = 0;                          // byte j: element e0 + j flips
    if (all_channels) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            lo |= w[j] < m.map_flip_p32 ? 1u << (8 * j) : 0u;
            hi |= w[4 + j] < m.map_flip_p32 ? 1u << (8 * j) : 0u;
        }
    } else {
        int c = e0 / plane, next = (c + 1) * plane;   // channel of element e, and its end
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            while (e0 + j >= next) { ++c; next += plane; }
            const uint32_t f = uint32_t(((m.map_channels >> c) & 1u) && w[j] < m.map_flip_p32);
            (j < 4 ? lo : hi) |= f << (8 * (j & 3));
        }
    }
    const uint64_t flips = uint64_t(lo) | (uint64_t(hi) << 32);
    if (whole) {
        const uint64_t low7 = 0x7F7F7F7F7F7F7F7Full;  // bit 7 of a byte: the byte is not 0
        const uint64_t set = ((((v & low7) + low7) | v) >> 7) & 0x0101010101010101ull;
        const uint64_t out = set ^ flips;
        __builtin_memcpy(d, &out, 8);
    } else {
        for (int j = 0; e0 + j < per; ++j)
            d[j] = uint8_t(s[j] != 0) ^ uint8_t((flips >> (8 * j)) & 1u);
    }
}

__device__ inline int8_t other_value(int8_t old, bool higher) {
    const int v = (old == -1 || old == 0) ? old : 1;
    return int8_t(higher ? (v == 1 ? 0 : 1) : (v == -1 ? 0 : -1));
}

// n / d by the host's recip_of(d): exact for n * (d - 1) < 2^32.
__device__ inline uint32_t div_by(uint32_t n, uint32_t recip) {
    return recip ? __umulhi(n, recip) : n;
}

// One thread per Philox block of four entries, and behind a set's eb entry blocks its rb blocks
// of four rewards.  Entry e = rio * pat + rest: the pattern's rows are consecutive bytes, so four
// entries of one pattern are loaded and stored as one word; the position of the first comes from
// two multiplications, the others' by counting up.
__global__ void __launch_bounds__(256) mutate_rules_kernel(
    const int32_t *shape, const int8_t *in_src, const int8_t *out_src, const int32_t *reward_src,
    int8_t *in_dst, int8_t *out_dst, int32_t *reward_dst, int s0, int ns, int R, int C1, int mh,
    int mw, int eb, int rb, uint32_t recip_cells, uint32_t recip_mw, MutateArgs m) {
    const uint32_t t = blockIdx.x * blockDim.x + threadIdx.x;
    const uint32_t blocks_per = uint32_t(eb) + uint32_t(rb);
    if (t >= uint32_t(ns) * blocks_per) return;
    const uint32_t ss = t / blocks_per;
    uint32_t blk = t - ss * blocks_per;
    const uint32_t s = uint32_t(s0) + ss;
    const bool rewards = blk >= uint32_t(eb);
    if (rewards) blk -= uint32_t(eb);
    uint32_t w[8];
    philox_words(m.seed, m.generation, s, rewards ? 3 : 2, blk, w);
    if (rewards) {
        // the number of values, 0 for all 2^32
        const uint32_t span = uint32_t(m.reward_hi) - uint32_t(m.reward_lo) + 1u;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int r = int(blk) * 4 + q;
            if (r >= R) break;
            const size_t at = size_t(s) * R + size_t(r);
            int32_t v = reward_src[at];
            if (w[2 * q] < m.reward_p32)
                v = int32_t(uint32_t(m.reward_lo) + (span ? w[2 * q + 1] % span : w[2 * q + 1]));
            reward_dst[at] = v;
        }
        return;
    }
    const uint32_t cells = uint32_t(mh) * uint32_t(mw), pat = uint32_t(C1) * cells;
    const uint32_t e0 = blk * 4;
    uint32_t rio = e0 / pat;
    const uint32_t rest = e0 - rio * pat;
    int c = int(div_by(rest, recip_cells));
    const uint32_t cell = rest - uint32_t(c) * cells;
    int i = int(div_by(cell, recip_mw));
    int j = int(cell) - i * mw;
    const size_t rule0 = size_t(s) * R;
    size_t rule = rule0 + (rio >> 1);
    int sh = shape[2 * rule], sw = shape[2 * rule + 1];
    // does element q change, if its pattern covers it; then to the next element
    auto changes = [&](int q) {
        const bool hit = i < sh && j < sw && ((m.entry_channels >> c) & 1u) && w[2 * q] < m.entry_p32;
        if (++j == mw) {
            j = 0;
            if (++i == mh) {
                i = 0;
                ++c;
            }
        }
        return hit;
    };
    if (rest + 4 <= pat) {
        const size_t at = rule * pat + rest;
        uint32_t v, out = 0;
        __builtin_memcpy(&v, (rio & 1u ? out_src : in_src) + at, 4);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            int8_t b = int8_t(v >> (8 * q));
            if (changes(q)) b = other_value(b, w[2 * q + 1] & 1u);
            out |= uint32_t(uint8_t(b)) << (8 * q);
        }
        __builtin_memcpy((rio & 1u ? out_dst : in_dst) + at, &out, 4);
        return;
    }
    const uint32_t sides = 2u * uint32_t(R);          // the set's patterns
    uint32_t left = pat - rest;                       // elements of this pattern from here on
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        if (left == 0) {                              // on to the next pattern
            if (++rio == sides) break;
            left = pat;
            c = i = j = 0;
            rule = rule0 + (rio >> 1);
            sh = shape[2 * rule];
            sw = shape[2 * rule + 1];
        }
        const size_t at = rule * pat + (pat - left);
        int8_t b = (rio & 1u ? out_src : in_src)[at];
        if (changes(q)) b = other_value(b, w[2 * q + 1] & 1u);
        (rio & 1u ? out_dst : in_dst)[at] = b;
        --left;
    }
}

// ceil(2^32 / d), or 0 for d = 1 (div_by).
uint32_t recip_of(uint32_t d) { return uint32_t(((uint64_t(1) << 32) + d - 1) / d); }

unsigned grid_for(int64_t threads) { return unsigned((threads + 255) / 256); }

}  // namespace

hipError_t launch_mutate_maps(const uint8_t *src, uint8_t *dst, int n, int C, int H, int W,
                              const MutateArgs &m, hipStream_t s) {
    const int per = C * H * W;                 // <= 31 * 64 * 64 in the batch API; any int here
    const int blocks_per = per / 8 + (per % 8 != 0);
    const int all = (~m.map_channels & uint32_t((uint64_t(1) << C) - 1)) == 0;
    // a grid row per individual where rounding its blocks up to whole workgroups idles at most
    // one lane in sixteen, which is what the scalar rounds give back
    const bool row = int64_t((blocks_per + 255) / 256) * 256 * 15 <= int64_t(blocks_per) * 16;
    int chunk = std::max(1, int((int64_t(1) << 30) / blocks_per));         // t fits 31 bits
    if (row) chunk = std::min(chunk, 65535);                               // rows of a grid
    for (int k0 = 0; k0 < n; k0 += chunk) {
        const int nk = std::min(chunk, n - k0);
        const int64_t threads = int64_t(nk) * blocks_per;
        if (row)
            hipLaunchKernelGGL(mutate_maps_kernel<true>, dim3(grid_for(blocks_per), nk), dim3(256),
                               0, s, src, dst, k0, nk, per, H * W, blocks_per, all, m);
        else
            hipLaunchKernelGGL(mutate_maps_kernel<false>, dim3(grid_for(threads)), dim3(256), 0, s,
                               src, dst, k0, nk, per, H * W, blocks_per, all, m);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_mutate_rules(int S, int R, int C, int mh, int mw, const int32_t *shape,
                               const int8_t *in_src, const int8_t *out_src,
                               const int32_t *reward_src, int8_t *in_dst, int8_t *out_dst,
                               int32_t *reward_dst, const MutateArgs &m, hipStream_t s) {
    if (int64_t(S) * R == 0) return hipSuccess;
    const int C1 = C + 1;
    const int per = R * 2 * C1 * mh * mw;     // <= 252 * 2 * 32 * 16 * 16
    const int eb = (per + 3) / 4, rb = (R + 3) / 4;
    const int chunk = std::max(1, int((int64_t(1) << 30) / (eb + rb)));
    for (int s0 = 0; s0 < S; s0 += chunk) {
        const int ns = std::min(chunk, S - s0);
        hipLaunchKernelGGL(mutate_rules_kernel, dim3(grid_for(int64_t(ns) * (eb + rb))), dim3(256),
                           0, s, shape, in_src, out_src, reward_src, in_dst, out_dst, reward_dst,
                           s0, ns, R, C1, mh, mw, eb, rb, recip_of(uint32_t(mh) * uint32_t(mw)),
                           recip_of(uint32_t(mw)), m);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace av
