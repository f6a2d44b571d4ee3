// Pieces shared by the kernels that hold one environment per wave in 16-lane groups (k_group.hip,
// k_solo.hip): the probe table's layout, merged input entries, rows next to a lane's own, and the
// exact write of a channel.
#pragma once

#include <type_traits>

#include "av_internal.h"

namespace av {

constexpr int kCountBits = 8;           // exact write counters: a channel list holds <= 254
                                        // entries (eligibility: rules x pattern cells <= 254)
constexpr int kHdrWords = int(sizeof(RuleHdr) / 4);
constexpr int kProbeEntries = 4;        // input entries of every rule tested in one round
constexpr int kProbeWords = 12;         // probe table row: entries 0-3, anchor word, match
                                        // offset | count << 16, vote offset | count << 16,
                                        // voted channels, entries 4-7
// Input entries merged per plane row: o | jb << 12 | care << 16 | want << 24 tests row
// o + y of the planes (o = c * PR + i: pattern row i of plane c) at the pattern columns
// 8 jb + j, j < 8, whose bit j of care is set: there the cell must equal bit j of want.
// kPassEntry tests no column (it passes everywhere).
constexpr uint32_t kPassEntry = 0u;
constexpr int kMaxEntryOffset = 4095;

// Words per plane row block: HR rows plus the pattern rows hanging below the last one,
// rounded up to 4 (16-byte aligned probe table after the planes).
__host__ __device__ constexpr int group_plane_words(int Hq, int max_pat_h) {
    return (Hq + max_pat_h - 1 + 3) & ~3;
}

__device__ inline uint32_t low_mask(int bits) { return bits >= 32 ? ~0u : ((1u << bits) - 1u); }

// Copy n words from global memory to LDS, eight loads of a lane in flight before its writes.
__device__ inline void copy_to_lds(uint32_t *dst, const uint32_t *src, int n, int lane) {
    for (int w0 = lane; w0 < n; w0 += 8 * 64) {
        uint32_t v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int w = w0 + 64 * u;
            v[u] = w < n ? src[w] : 0u;
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int w = w0 + 64 * u;
            if (w < n) dst[w] = v[u];
        }
    }
}

// Does any lane of this lane's group hold a nonzero?
template <int Hq>
__device__ inline bool group_any(bool p, int lane) {
    const unsigned long long bal = __builtin_amdgcn_ballot_w64(p);
    if (Hq >= 64) return bal != 0ull;
    const int base = lane & ~(Hq - 1);
    return ((bal >> base) & ((1ull << Hq) - 1ull)) != 0ull;
}

// Rows y + 1 (next) and y - 1 (prev) of the rows a lane holds, 0 past the group's ends, RPL
// of them (2: on maps of 17 to 32 rows a lane of a 16-lane group holds rows y and y + 16):
// within each 16-row half a DPP row shift, across the halves a DPP row rotate (lane 15's next
// row is lane 0's second row, lane 0's second row's previous row is lane 15's first).
template <int Hq, int RPL>
__device__ inline void next_rows(const uint32_t (&v)[RPL], uint32_t (&n)[RPL], int lane, int y) {
    static_assert(Hq == 16, "16-lane groups");
    (void)lane;
    if constexpr (RPL == 1) {
        n[0] = uint32_t(__builtin_amdgcn_update_dpp(0, int(v[0]), 0x101, 0xF, 0xF, true));
    } else {
        const uint32_t s0 = uint32_t(__builtin_amdgcn_update_dpp(0, int(v[0]), 0x101, 0xF, 0xF, true));
        const uint32_t w1 = uint32_t(__builtin_amdgcn_update_dpp(0, int(v[1]), 0x12F, 0xF, 0xF, true));
        n[0] = y == Hq - 1 ? w1 : s0;
        n[1] = uint32_t(__builtin_amdgcn_update_dpp(0, int(v[1]), 0x101, 0xF, 0xF, true));
    }
}
template <int Hq, int RPL>
__device__ inline void prev_rows(const uint32_t (&v)[RPL], uint32_t (&p)[RPL], int lane, int y) {
    static_assert(Hq == 16, "16-lane groups");
    (void)lane;
    if constexpr (RPL == 1) {
        (void)y;
        p[0] = uint32_t(__builtin_amdgcn_update_dpp(0, int(v[0]), 0x111, 0xF, 0xF, true));
    } else {
        p[0] = uint32_t(__builtin_amdgcn_update_dpp(0, int(v[0]), 0x111, 0xF, 0xF, true));
        const uint32_t t1 = uint32_t(__builtin_amdgcn_update_dpp(0, int(v[1]), 0x111, 0xF, 0xF, true));
        const uint32_t w0 = uint32_t(__builtin_amdgcn_update_dpp(0, int(v[0]), 0x121, 0xF, 0xF, true));
        p[1] = y == 0 ? w0 : t1;
    }
}

template <int RPL>
__device__ inline bool any_row(const uint32_t (&v)[RPL]) {
    uint32_t o = 0u;
#pragma unroll
    for (int h = 0; h < RPL; ++h) o |= v[h];
    return o != 0u;
}

// Count the votes of rule r's channel-list entries lo .. hi - 1 (packed r | i << 8 | j << 16 |
// plus << 24) into the KB-bit bit-sliced counters cnt of the lane's rows yr: a plus vote adds
// its cells, a minus vote adds the complement of its cells; nm counts the minus entries.  Four
// entries at a time: carry-save adders make the four one-bit planes a 3-bit number, then one
// ripple add.
template <int KB, int RPL>
__device__ inline void count_votes(uint32_t (&cnt)[RPL][KB], int &nm, const uint32_t *vl, int lo,
                                   int hi, const uint32_t *Mr, const int (&yr)[RPL],
                                   const bool (&rw)[RPL]) {
    for (int ev = lo; ev < hi; ev += 4) {
        uint32_t v[4];
        bool live[4], minus[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = vl[min(ev + u, hi - 1)];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            live[u] = ev + u < hi;
            minus[u] = live[u] && !((v[u] >> 24) & 1u);
            nm += minus[u] ? 1 : 0;
        }
#pragma unroll
        for (int h = 0; h < RPL; ++h) {
            uint32_t x[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const uint32_t t =
                    rw[h] ? Mr[yr[h] - int((v[u] >> 8) & 255u)] << ((v[u] >> 16) & 255u) : 0u;
                x[u] = !live[u] ? 0u : minus[u] ? ~t : t;
            }
            const uint32_t a = x[0] ^ x[1], s1 = a ^ x[2];
            const uint32_t c1 = (x[0] & x[1]) | (x[2] & a);            // weight 2
            const uint32_t s0 = s1 ^ x[3], c2 = s1 & x[3];             // weight 1, 2
            const uint32_t w2 = c1 ^ c2, w4 = c1 & c2;                 // weight 2, 4
            uint32_t *const q = cnt[h];
            uint32_t k = q[0] & s0;
            q[0] ^= s0;
            const uint32_t a1 = q[1] ^ w2;
            const uint32_t k1 = (q[1] & w2) | (k & a1);
            q[1] = a1 ^ k;
            const uint32_t a2 = q[2] ^ w4;
            k = (q[2] & w4) | (k1 & a2);
            q[2] = a2 ^ k1;
#pragma unroll
            for (int b = 3; b < KB; ++b) {
                const uint32_t kq = q[b] & k;
                q[b] ^= k;
                k = kq;
            }
        }
    }
}

// The exact write of channel c for the lane's rows (needed only where some cell of the group
// got votes of both signs): the votes on c of every rule in `fired` (the channel's vote list
// `vl`, ordered by rule; rule r's entries are vl[rsc[r] & 0xFFFF .. rsc[r] >> 16)) with the old
// value as a plus vote.  One counter takes old + #plus + (#minus entries - #minus votes), so a
// cell is set, old + #plus - #minus >= 1, where it reaches 1 + #minus entries.  A list holds
// at most 254 entries (eligibility: every entry is a distinct rule and pattern cell), so
// 8-bit counters never overflow; 4 bits do when the fired rules' entries are at most 14.
// With `moves` (the player plane) the four moves' votes, two entries each (-1 on the player's
// cell, +1 on the cell it moves to), are read from their match rows at once: the counter starts
// at old + their four plus votes + (4 - their four minus votes) and only the loaded rules'
// lists are walked.  (The four-wave kernels of groups of up to two rules, whose probe rows stay
// in registers, walk the moves too: the start's registers would spill the step's own.)
template <int RPL>
__device__ inline void exact_channel(const uint32_t (&old)[RPL], uint64_t fired, bool moves,
                                     const uint32_t *vl, const uint32_t *rsc, const uint32_t *M,
                                     int MS, int pad, const int (&yr)[RPL], const bool (&rw)[RPL],
                                     uint32_t (&out)[RPL]) {
    const uint64_t walk = moves ? fired & ~((1ull << kMoveRules) - 1ull) : fired;
    int total = moves ? 2 * kMoveRules : 0;
    for (uint64_t fr = walk; fr; fr &= fr - 1) {
        const uint32_t rs = rsc[__builtin_ctzll(fr)];
        total += int(rs >> 16) - int(rs & 0xFFFFu);
    }
    int nm = moves ? kMoveRules : 0;
    auto ge = [&](auto &cnt, auto kb) {           // cnt >= 1 + nm, bit-sliced
        constexpr int KB = decltype(kb)::value;
        const uint32_t T = uint32_t(1 + nm);
#pragma unroll
        for (int h = 0; h < RPL; ++h) {
            uint32_t gt = 0u, eq = ~0u;
#pragma unroll
            for (int q = KB - 1; q >= 0; --q) {
                const uint32_t tb = ((T >> q) & 1u) ? ~0u : 0u;
                gt |= eq & cnt[h][q] & ~tb;
                eq &= ~(cnt[h][q] ^ tb);
            }
            out[h] = gt | eq;
        }
    };
    auto run = [&](auto kb) {
        constexpr int KB = decltype(kb)::value;
        uint32_t cnt[RPL][KB];
#pragma unroll
        for (int h = 0; h < RPL; ++h) {
#pragma unroll
            for (int q = 0; q < KB; ++q) cnt[h][q] = 0u;
            const uint32_t o = rw[h] ? old[h] : 0u;
            if (moves) {
                // match rows of right, left, down, up (rules 0..3) at this row and the one above
                const uint32_t *m = M + pad + yr[h];
                const uint32_t m0 = m[0], m1 = m[MS], m2 = m[2 * MS], m3 = m[3 * MS];
                const uint32_t m2p = m[2 * MS - 1], m3p = m[3 * MS - 1];
                const uint32_t a1 = m0 << 1, b2 = m1 << 1;
                // plus: old, a1, m1, m2p, m3 -> p2 p1 p0
                const uint32_t s1 = o ^ a1 ^ m1, c1 = (o & a1) | (m1 & (o ^ a1));
                const uint32_t p0 = s1 ^ m2p ^ m3, c2 = (s1 & m2p) | (m3 & (s1 ^ m2p));
                const uint32_t p1 = c1 ^ c2, p2 = c1 & c2;
                // complements of the minus votes m0, b2, m2, m3p -> q2 q1 q0 (4 - their sum)
                const uint32_t s3 = m0 ^ b2 ^ m2, c3 = (m0 & b2) | (m2 & (m0 ^ b2));
                const uint32_t q0 = s3 ^ m3p, q1 = c3 ^ (s3 | m3p), q2 = ~(c3 | s3 | m3p);
                // p + q (at most 9)
                const uint32_t k0 = p0 & q0;
                const uint32_t k1 = (p1 & q1) | (k0 & (p1 ^ q1));
                const uint32_t k2 = (p2 & q2) | (k1 & (p2 ^ q2));
                cnt[h][0] = p0 ^ q0;
                cnt[h][1] = p1 ^ q1 ^ k0;
                cnt[h][2] = p2 ^ q2 ^ k1;
                cnt[h][3] = k2;
            } else {
                cnt[h][0] = o;
            }
        }
        for (uint64_t fr = walk; fr; fr &= fr - 1) {
            const int r = __builtin_ctzll(fr);
            const uint32_t rs = rsc[r];
            count_votes<KB, RPL>(cnt, nm, vl, int(rs & 0xFFFFu), int(rs >> 16),
                                 M + r * MS + pad, yr, rw);
        }
        ge(cnt, kb);
    };
    if (total <= 14) run(std::integral_constant<int, 4>{});
    else run(std::integral_constant<int, kCountBits>{});
}

}  // namespace av
