// wave engine, one-wave form: sequential rule order and rule application control on maps of up to
// 32 x 32.
//
// One environment per wave and one wave per workgroup, so a step meets no barrier: the wave's LDS
// operations take effect in the order it issues them.  The wave's 64 lanes form four groups of 16;
// lane y of every group holds map row y and, on maps of 17 to 32 rows, row y + 16 too.  Rules are
// dealt to the groups as they come up, not by index: a window of eight rules is probed at once
// (two per group, each with its first four merged entries), and the rules that pass are finished
// four at a time, one per group, so a group never waits for another group's list.
//
// What bounds it: a step is a chain of dependent LDS round trips (probe row, plane rows, the rest
// of a candidate's entries, votes, write), with one to four waves per SIMD to hide them.  The
// multi-wave form (k_wave.hip) spends those steps at barriers instead: two per rule in sequential
// order, and with control up to fifteen per fired rule.
//
// LDS (32-bit rows; PR, HR, the probe table and the merged entries as in k_group.hip):
//   P    [C+1][PR]     the map and the force plane (channel C)
//   M    [R+4][PR]     match planes, row y at ph - 1 + y
//   PL, MI [NC][HR]    per channel, the OR of the +1 and of the -1 votes (NC: C, or C + 1 in
//                      sequential order, where later rules read the force plane)
//   I0   [C][HR]       the initial rows, for resets
//   PT   [R+5][12]     probe table; RS [NC][R+4] rule ranges of the channel vote lists, RM [NC][2]
//   CT   [R+4][3]      control: the rule's cap and its inhibitors' mask
//   KEY  [H][W|1]      random site order: the step's index channel
//   program            (when it fits) headers, merged entries, rule-major and channel-major votes
//
// Per step (paper Sec. 2.1, Sec. 2.1.1, Sec. 2.2.1), parallel rule order:
//   force, moves       in registers;
//   probe, match       every loaded rule on the same map; a fired rule leaves its match plane in M;
//   control            the fired rules in index order: matches whose patch overlaps an applied
//                      match of an inhibiting rule are dropped, then at most `cap` are kept, those
//                      first in row-major order or with the largest keys (below);
//   votes, write       four votes of a rule per group and round; then every voted channel.
// Sequential rule order: the moves one after another in registers; then, from the first rule on,
// the rules of a window are matched against the map as it is, and only the first one that applies
// (after its control) writes: every rule before it did not match that map, and the search goes on
// behind it on the new map.  The result is that of applying every rule in turn, at one round per
// rule that fires instead of one per rule.
//
// A cap in random order: every lane takes eight cells of each of its rows (cells 8 g + i of group
// g) and holds their keys, 0 where the rule does not match (a key is never 0: its low bits are the
// rank 4095 - pos, and pos is at most 1023), so the wave holds every match's key in registers.
// A threshold T with exactly `cap` keys at or above it is found bit by bit from the top (one
// ballot per held key and bit); keys never tie, and with keys drawn at random the count meets
// `cap` after about log2(matches) bits.
#include <algorithm>

#include "group_common.h"
#include "philox.h"

namespace av {
namespace {

constexpr int kHq = 16;                 // lanes of a group
constexpr int kG = 4;                   // groups of a wave
constexpr int kCellsPerLane = 8;        // cells of a row one lane holds keys for (32 / kG)
constexpr int kProgLdsSteps = 16;       // launches of fewer steps read the program from memory

__host__ __device__ constexpr int key_stride(int W) { return W | 1; }

// Inclusive prefix sum over the 16 lanes of a group.
__device__ inline int group_prefix(int v) {
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, true);   // row_shr:1
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, true);
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, true);
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, true);
    return v;
}

// OR over the four groups (lanes y, y + 16, y + 32, y + 48).
__device__ inline uint32_t groups_or(uint32_t v) {
    const auto p = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    v = p[0] | p[1];
    const auto q = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    return q[0] | q[1];
}

// Orders the wave's LDS writes before its later LDS reads for the compiler (the hardware keeps
// a wave's LDS operations in order, and no instruction comes of it).
__device__ inline void lds_order() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
}

__device__ inline uint32_t uniform(uint32_t v) {
    return uint32_t(__builtin_amdgcn_readfirstlane(int(v)));
}

template <int RPL, int NJ, bool SEQ, bool CTL, bool PROG_LDS>
__global__ void __launch_bounds__(64, 2) solo_step(StepArgs a) {
    constexpr int HR = kHq * RPL;
    extern __shared__ __align__(16) uint32_t lds[];
    const int lane = int(threadIdx.x), g = lane / kHq, y = lane % kHq;
    const uint64_t t_start = __builtin_amdgcn_s_memtime();
    const int b = a.order ? a.order[blockIdx.x] : int(blockIdx.x);
    const int H = a.H, W = a.W, C = a.C, C1 = C + 1, Rt = a.prog.rules_per_set;
    const int NC = SEQ ? C1 : C;
    const int PAD = a.max_pat_h - 1;
    const int PR = group_plane_words(HR, a.max_pat_h), MS = PR;
    const int s = a.per_env ? b : 0;
    const int nl = Rt - kMoveRules;               // loaded rules
    int yr[RPL];
    bool rw[RPL];
#pragma unroll
    for (int h = 0; h < RPL; ++h) {
        yr[h] = y + kHq * h;
        rw[h] = yr[h] < H;
    }
    const uint32_t wmask = low_mask(W);

    uint32_t *P = lds;                             // [C1][PR]
    uint32_t *M = P + C1 * PR;                     // [Rt][MS]
    uint32_t *PL = M + Rt * MS;                    // [NC][HR]
    uint32_t *MI = PL + NC * HR;                   // [NC][HR]
    uint32_t *I0 = MI + NC * HR;                   // [C][HR]
    uint32_t *PT = I0 + C * HR;                    // [Rt + 1][kProbeWords]
    uint32_t *RS = PT + (Rt + 1) * kProbeWords;    // [NC][Rt]
    uint32_t *RM = RS + NC * Rt;                   // [NC][2]
    uint32_t *CT = RM + 2 * NC;                    // [Rt][3] (CTL)
    uint32_t *KEY = CT + (CTL ? 3 * Rt : 0);       // [H][key_stride(W)] (random order)
    uint32_t *lprog = KEY + (CTL && a.ctl.random ? H * key_stride(W) : 0);

    const uint32_t *ghdr = reinterpret_cast<const uint32_t *>(a.prog.hdr + size_t(s) * Rt);
    const uint32_t *gment = a.prog.gmatch + size_t(s) * a.prog.gmatch_stride;
    const uint32_t *gvent = a.prog.rvote + size_t(s) * a.prog.rvote_stride;
    const uint32_t *gvl = reinterpret_cast<const uint32_t *>(a.prog.votes + size_t(s) * C1);
    const uint32_t *gvote = a.prog.vote + size_t(s) * a.prog.vote_stride;
    const int hdr_words = Rt * kHdrWords;
    const uint32_t *hdrw = ghdr, *ment = gment, *vent = gvent, *vlw = gvl, *vote = gvote;
    if constexpr (PROG_LDS) {
        uint32_t *ph = lprog, *pm = ph + hdr_words, *pv = pm + a.prog.gmatch_stride;
        uint32_t *pl = pv + a.prog.rvote_stride, *pc = pl + 2 * C1;
        copy_to_lds(ph, ghdr, hdr_words, lane);
        copy_to_lds(pm, gment, a.prog.gmatch_stride, lane);
        copy_to_lds(pv, gvent, a.prog.rvote_stride, lane);
        copy_to_lds(pl, gvl, 2 * C1, lane);
        copy_to_lds(pc, gvote, a.prog.vote_stride, lane);
        hdrw = ph;
        ment = pm;
        vent = pv;
        vlw = pl;
        vote = pc;
    }
    {
        const int words = C1 * PR + Rt * MS + (2 * NC + C) * HR;   // (PT, RS and RM are copied)
        for (int w = lane; w < words; w += 64) lds[w] = 0u;
    }
    copy_to_lds(PT, a.prog.gtab + size_t(s) * a.prog.gtab_stride, a.prog.gtab_stride, lane);
    if constexpr (CTL) {
        for (int r = lane; r < Rt; r += 64) {
            const size_t cr = size_t(s) * Rt + r;
            CT[3 * r] = uint32_t(a.ctl.limit[cr]);
            CT[3 * r + 1] = a.ctl.inhibit[cr * a.ctl.words];
            CT[3 * r + 2] = a.ctl.words > 1 ? a.ctl.inhibit[cr * a.ctl.words + 1] : 0u;
        }
    }
    // lane l takes row l % H of channels l / H, l / H + 64 / H, ...
    {
        const int rcs = 64 / H, rcl = lane / H, rrow = lane - rcl * H;
        auto load_rows = [&](const auto *st, const auto *in) {
            for (int c = rcl; c < C; c += rcs) {
                const size_t at = (size_t(c) * a.B + b) * H + rrow;
                P[c * PR + rrow] = uint32_t(st[at]);
                I0[c * HR + rrow] = uint32_t(in[at]);
            }
        };
        if (rcl < rcs) {
            if (a.row_bytes == 2)
                load_rows(static_cast<const uint16_t *>(a.state), static_cast<const uint16_t *>(a.init));
            else
                load_rows(static_cast<const uint32_t *>(a.state), static_cast<const uint32_t *>(a.init));
        }
    }
    __syncthreads();   // (one wave: orders the set-up's LDS writes before the step's reads)
    int t_env = a.t[b];
    const uint64_t nbase = a.nctr[b];

    auto miss = [&](uint32_t e, uint32_t (&bad)[RPL]) {
        uint32_t v[RPL];
#pragma unroll
        for (int h = 0; h < RPL; ++h) {
            v[h] = P[int(e & uint32_t(kMaxEntryOffset)) + yr[h]];
            if constexpr (NJ > 3) v[h] >>= (e >> 9) & 24u;
        }
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            const uint32_t want = uint32_t(int32_t(e << (7 - j)) >> 31);
            const uint32_t care = uint32_t(int32_t(e << (15 - j)) >> 31);
#pragma unroll
            for (int h = 0; h < RPL; ++h) bad[h] |= ((v[h] >> j) ^ want) & care;
        }
    };
    auto entries4 = [&](uint32_t e0, uint32_t e1, uint32_t e2, uint32_t e3, uint32_t (&m)[RPL]) {
        uint32_t bad[RPL];
#pragma unroll
        for (int h = 0; h < RPL; ++h) bad[h] = 0u;
        miss(e0, bad);
        miss(e1, bad);
        miss(e2, bad);
        miss(e3, bad);
#pragma unroll
        for (int h = 0; h < RPL; ++h) m[h] &= ~bad[h];
    };
    // probe of loaded rules w .. w + 7 on the current map, rule w + 4 q + g by group g; the match
    // rows so far go to M; returns the mask of those that hold an anchor (bit 4 q + g)
    auto probe = [&](int w) -> uint32_t {
        uint32_t m[2][RPL];
        uint4 e[2];
        uint32_t pv[2];
        const int i0 = w + g, i1 = w + 4 + g;
        const int r0 = i0 < nl ? kMoveRules + i0 : Rt, r1 = i1 < nl ? kMoveRules + i1 : Rt;
        e[0] = *reinterpret_cast<const uint4 *>(PT + r0 * kProbeWords);   // (row Rt: no anchors)
        e[1] = *reinterpret_cast<const uint4 *>(PT + r1 * kProbeWords);
        pv[0] = PT[r0 * kProbeWords + 4];
        pv[1] = PT[r1 * kProbeWords + 4];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
#pragma unroll
            for (int h = 0; h < RPL; ++h)
                m[q][h] = yr[h] < int(pv[q] >> 8) ? ~0u >> (pv[q] & 255u) : 0u;
            entries4(e[q].x, e[q].y, e[q].z, e[q].w, m[q]);
        }
        uint32_t cand = 0u;
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int r = q ? r1 : r0;
            if (r < Rt) {
#pragma unroll
                for (int h = 0; h < RPL; ++h) M[r * MS + PAD + yr[h]] = m[q][h];
            }
            const unsigned long long bal = __builtin_amdgcn_ballot_w64(any_row<RPL>(m[q]));
#pragma unroll
            for (int gg = 0; gg < kG; ++gg)
                cand |= ((bal >> (kHq * gg)) & 0xFFFFull) ? 1u << (4 * q + gg) : 0u;
        }
        lds_order();
        return cand;
    };
    // the rest of the entries of up to four candidates (rule indices c0 .. c3, Rt: none), one per
    // group; the final match rows go to M; returns the mask of the groups whose rule fired
    auto finish = [&](int c0, int c1, int c2, int c3) -> uint32_t {
        const int r = g == 0 ? c0 : g == 1 ? c1 : g == 2 ? c2 : c3;
        const bool live = r < Rt;
        const uint32_t meta = PT[r * kProbeWords + 5];
        const uint4 q = *reinterpret_cast<const uint4 *>(PT + r * kProbeWords + 8);
        uint32_t m[RPL];
#pragma unroll
        for (int h = 0; h < RPL; ++h) m[h] = live ? M[(live ? r : 0) * MS + PAD + yr[h]] : 0u;
        const int off = int(meta & 0xFFFFu), cnt = live ? int(meta >> 16) : 0, last = cnt - 1;
        uint32_t x[4] = {q.x, q.y, q.z, q.w};
        for (int e = kProbeEntries;; e += 4) {
            const bool more = e < cnt && any_row<RPL>(m);
            if (!__builtin_amdgcn_ballot_w64(more)) break;
            uint32_t nx[4];
            const bool next = e + 4 < cnt;        // (reads stay inside the rule's entries)
#pragma unroll
            for (int u = 0; u < 4; ++u) nx[u] = next ? ment[off + min(e + 4 + u, last)] : kPassEntry;
            entries4(more ? x[0] : kPassEntry, more ? x[1] : kPassEntry, more ? x[2] : kPassEntry,
                     more ? x[3] : kPassEntry, m);
#pragma unroll
            for (int u = 0; u < 4; ++u) x[u] = nx[u];
        }
        if (live) {
#pragma unroll
            for (int h = 0; h < RPL; ++h) M[r * MS + PAD + yr[h]] = m[h];
        }
        const unsigned long long bal = __builtin_amdgcn_ballot_w64(any_row<RPL>(m));
        uint32_t f = 0u;
#pragma unroll
        for (int gg = 0; gg < kG; ++gg) f |= ((bal >> (kHq * gg)) & 0xFFFFull) ? 1u << gg : 0u;
        lds_order();
        return f;
    };

    uint32_t have_keys = 0u;                      // (random order) passes of 64 blocks in KEY
    // control of rule r, which fired on this step's map: drops inhibited matches (inhibitors among
    // `applied`) and those above the cap; false when none is left.  Every group does the same
    // work on all rows, but for the keys, which are split over the groups.
    auto control = [&](int r, uint64_t applied, uint64_t n) -> bool {
        uint32_t acc[RPL];
#pragma unroll
        for (int h = 0; h < RPL; ++h) acc[h] = M[r * MS + PAD + yr[h]];
        const int lim = int(uniform(CT[3 * r]));
        const uint32_t pv = uniform(PT[r * kProbeWords + 4]);
        const int hn = H + 1 - int(pv >> 8), hm = W - 31 + int(pv & 255u);
        uint64_t inh = (uint64_t(uniform(CT[3 * r + 1])) | (uint64_t(uniform(CT[3 * r + 2])) << 32)) & applied;
        for (; inh; inh &= inh - 1) {
            const int q = __builtin_ctzll(inh);
            const uint32_t qv = uniform(PT[q * kProbeWords + 4]);
            const int nq = H + 1 - int(qv >> 8), mq = W - 31 + int(qv & 255u);
            const uint32_t *Mq = M + q * MS + PAD;
            uint32_t o[RPL];
#pragma unroll
            for (int h = 0; h < RPL; ++h) o[h] = 0u;
            // anchors of q whose patch meets an hn-row patch at the lane's row (rows above the map
            // are zero rows of M, the last row stands for those below it)
            for (int d = 1 - nq; d < hn; ++d) {
#pragma unroll
                for (int h = 0; h < RPL; ++h) o[h] |= Mq[min(yr[h] + d, HR - 1)];
            }
#pragma unroll
            for (int h = 0; h < RPL; ++h) {
                uint32_t dil = o[h];
                for (int d = 1; d < hm; ++d) dil |= o[h] >> d;
                for (int d = 1; d < mq; ++d) dil |= o[h] << d;
                acc[h] &= ~dil;
            }
        }
        if (lim > 0) {
            int inc[RPL], total = 0;              // matches up to and including the lane's rows
#pragma unroll
            for (int h = 0; h < RPL; ++h) {
                inc[h] = group_prefix(__popc(acc[h])) + total;
                total = __builtin_amdgcn_readlane(inc[h], kHq - 1);
            }
            if (total > lim) {
                if (!a.ctl.random) {
#pragma unroll
                    for (int h = 0; h < RPL; ++h) {
                        // drop the row's last matches past the cap
                        for (int over = min(inc[h] - lim, __popc(acc[h])); over > 0; --over)
                            acc[h] &= ~(0x80000000u >> __builtin_clz(acc[h]));
                    }
                } else {
                    // the keys of 512 cells per pass of the wave, made when first needed
                    const int passes = (H * W + 511) / 512;
                    for (int p = 0; p < passes; ++p) {
                        if ((have_keys >> p) & 1u) continue;
                        const int gi = 64 * p + lane;
                        if (gi * 8 < H * W) {
                            uint32_t u[8];
                            philox_words(a.ctl.seed, n, uint64_t(b), 0, uint64_t(gi), u);
                            int ky = (gi * 8) / W, kx = gi * 8 - ky * W;
#pragma unroll
                            for (int j = 0; j < 8; ++j) {
                                if (gi * 8 + j < H * W)
                                    KEY[ky * key_stride(W) + kx] =
                                        (u[j] & 0xFFFFF000u) | uint32_t(4095 - (gi * 8 + j));
                                ++kx;
                                if (kx == W) { kx = 0; ++ky; }
                            }
                        }
                    }
                    have_keys = (1u << passes) - 1u;
                    lds_order();
                    uint32_t key[RPL][kCellsPerLane];
#pragma unroll
                    for (int h = 0; h < RPL; ++h) {
#pragma unroll
                        for (int i = 0; i < kCellsPerLane; ++i) {
                            const int x = kCellsPerLane * g + i;
                            const bool on = (acc[h] >> x) & 1u;
                            key[h][i] = on ? KEY[yr[h] * key_stride(W) + x] : 0u;
                        }
                    }
                    // the largest T with at least lim keys >= T, bit by bit; exactly lim ends it
                    uint32_t T = 0u;
                    for (int bit = 31; bit >= 0; --bit) {
                        const uint32_t t = T | (1u << bit);
                        int at_least = 0;
#pragma unroll
                        for (int h = 0; h < RPL; ++h)
#pragma unroll
                            for (int i = 0; i < kCellsPerLane; ++i)
                                at_least += __popcll(__builtin_amdgcn_ballot_w64(key[h][i] >= t));
                        if (at_least >= lim) T = t;
                        if (at_least == lim) break;
                    }
                    // each group's kept cells, OR-ed over the groups
#pragma unroll
                    for (int h = 0; h < RPL; ++h) {
                        uint32_t keep = 0u;
#pragma unroll
                        for (int i = 0; i < kCellsPerLane; ++i)
                            keep |= key[h][i] >= T ? 1u << (kCellsPerLane * g + i) : 0u;
                        acc[h] = groups_or(keep);
                    }
                }
            }
        }
#pragma unroll
        for (int h = 0; h < RPL; ++h) M[r * MS + PAD + yr[h]] = acc[h];
        lds_order();
        return __builtin_amdgcn_ballot_w64(any_row<RPL>(acc)) != 0ull;
    };

    uint32_t ablk = 0u;     // lane l: action of step k0 + l of the current block of 64
    float rbuf = 0.f;       // lane l: reward of step k0 + l
    uint32_t dbuf = 0u;     // lane l: done flag of step k0 + l
    uint32_t *const F = P + C * PR;
    uint32_t *const P2 = P + kChPlayer * PR;
    const uint32_t cm1 = low_mask(W - 1);         // anchors of a 1 x 2 pattern
    uint32_t vrow2[RPL];                          // rows of a 2 x 1 pattern's anchors
#pragma unroll
    for (int h = 0; h < RPL; ++h) vrow2[h] = (yr[h] + 2 <= H) ? wmask : 0u;
    // the player and wall rows of the lane (every group holds them), 0 past the map
    uint32_t Py[RPL], Wy[RPL];
#pragma unroll
    for (int h = 0; h < RPL; ++h) {
        Py[h] = rw[h] ? P2[yr[h]] : 0u;
        Wy[h] = rw[h] ? P[kChWall * PR + yr[h]] : 0u;
    }

    for (int k = 0; k < a.k; ++k) {
        const int kb = k & 63;
        if (kb == 0) ablk = (k + lane < a.k) ? uint32_t(a.actions[size_t(k + lane) * a.B + b]) : 0u;
        const int act = __builtin_amdgcn_readlane(int(ablk), kb);
        if constexpr (CTL) have_keys = 0u;
        uint32_t Pn[RPL], Wn[RPL], Pp[RPL], Fy[RPL], Fn[RPL];
        next_rows<kHq, RPL>(Py, Pn, lane, y);
        next_rows<kHq, RPL>(Wy, Wn, lane, y);
        prev_rows<kHq, RPL>(Py, Pp, lane, y);
#pragma unroll
        for (int h = 0; h < RPL; ++h)
            Fy[h] = act == 1 ? Pn[h] : act == 3 ? Pp[h] : act == 2 ? ((Py[h] << 1) & wmask)
                  : act == 4 ? (Py[h] >> 1) : 0u;

        int rsum = 0;                             // (lanes of group 0)
        uint32_t lvoted = 0u;                     // channels the loaded rules voted on
        // the votes of rule r's match rows (M), four per group and round, and its reward
        auto cast = [&](int r) {
            const uint32_t pvw = PT[r * kProbeWords + 6];
            const int voff = int(pvw & 0xFFFFu), vcnt = int(pvw >> 16), vlast = vcnt - 1;
            const uint32_t *ve = vent + voff;
            const uint32_t *Mr = M + r * MS + PAD;
            uint32_t v[4];
            if (vcnt > 0) {
#pragma unroll
                for (int u = 0; u < 4; ++u) v[u] = ve[min(g + 4 * u, vlast)];
            }
            for (int ev = 0; ev < vcnt; ev += 4 * kG) {
                uint32_t cv[4], tv[4][RPL];
#pragma unroll
                for (int u = 0; u < 4; ++u) cv[u] = v[u];
                if (ev + 4 * kG < vcnt) {
#pragma unroll
                    for (int u = 0; u < 4; ++u) v[u] = ve[min(ev + 4 * kG + g + 4 * u, vlast)];
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) {
#pragma unroll
                    for (int h = 0; h < RPL; ++h)
                        tv[u][h] = Mr[yr[h] - int((cv[u] >> 8) & 255u)] << ((cv[u] >> 16) & 255u);
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) {
#pragma unroll
                    for (int h = 0; h < RPL; ++h)
                        if (rw[h] && tv[u][h])
                            atomicOr(((cv[u] >> 24) & 1u ? PL : MI) + int(cv[u] & 255u) * HR + yr[h],
                                     tv[u][h]);
                }
            }
            const int reward = int(uniform(hdrw[r * kHdrWords + 2]));
            if (reward && g == 0) {
#pragma unroll
                for (int h = 0; h < RPL; ++h) rsum += reward * __popc(Mr[yr[h]]);
            }
            lvoted |= uniform(PT[r * kProbeWords + 7]);
            lds_order();
        };
        // new rows of the loaded rules' voted channels in `which`, group g taking every fourth
        // channel; pl0, mi0: the moves' votes on the player plane (parallel order)
        auto write = [&](uint32_t which, uint64_t fired, const uint32_t (&pl0)[RPL],
                         const uint32_t (&mi0)[RPL]) {
            // group g takes the g-th, (g + 4)-th, ... channel of `which`
            uint32_t left = which;
            while (left) {
                int c = -1;
#pragma unroll
                for (int gg = 0; gg < kG; ++gg) {
                    const int cg = left ? __builtin_ctz(left) : -1;
                    if (left) left &= left - 1u;
                    c = g == gg ? cg : c;
                }
                if (c < 0) continue;
                uint32_t old[RPL], nw[RPL], mixed = 0u;
#pragma unroll
                for (int h = 0; h < RPL; ++h) {
                    old[h] = P[c * PR + yr[h]];
                    uint32_t pl = PL[c * HR + yr[h]], mi = MI[c * HR + yr[h]];
                    if (!SEQ && c == kChPlayer) {
                        pl |= pl0[h];
                        mi |= mi0[h];
                    }
                    nw[h] = (old[h] | pl) & ~mi;
                    mixed |= pl & mi;
                    PL[c * HR + yr[h]] = 0u;
                    MI[c * HR + yr[h]] = 0u;
                }
                if (group_any<kHq>(mixed != 0u, lane))
                    exact_channel<RPL>(old, fired & (uint64_t(RM[2 * c]) | uint64_t(RM[2 * c + 1]) << 32),
                                       !SEQ && c == kChPlayer, vote + int(vlw[2 * c]), RS + c * Rt, M,
                                       MS, PAD, yr, rw, nw);
#pragma unroll
                for (int h = 0; h < RPL; ++h)
                    if (rw[h]) P[c * PR + yr[h]] = nw[h];
            }
            lds_order();
        };

        if constexpr (SEQ) {
            // the moves one after another: right, left, down, up (each takes the player from its
            // cell to the force cell next to it and consumes the force; a cell that a player
            // leaves and another enters keeps its tile: 1 + 1 - 1)
            auto any = [&](const uint32_t (&m)[RPL]) {
                return __builtin_amdgcn_ballot_w64(any_row<RPL>(m)) != 0ull;
            };
            bool moved = false;
            if (act >= 1 && act <= 4) {
                uint32_t m[RPL], mp[RPL];
#pragma unroll
                for (int h = 0; h < RPL; ++h) m[h] = Py[h] & (Fy[h] >> 1) & ~(Wy[h] >> 1) & cm1;
                if (any(m)) {
                    moved = true;
#pragma unroll
                    for (int h = 0; h < RPL; ++h) {
                        Py[h] = (Py[h] & ~m[h]) | (m[h] << 1);
                        Fy[h] &= ~(m[h] << 1);
                    }
                }
#pragma unroll
                for (int h = 0; h < RPL; ++h) m[h] = Fy[h] & ~Wy[h] & (Py[h] >> 1) & cm1;
                if (any(m)) {
                    moved = true;
#pragma unroll
                    for (int h = 0; h < RPL; ++h) {
                        Py[h] = (Py[h] & ~(m[h] << 1)) | m[h];
                        Fy[h] &= ~m[h];
                    }
                }
                next_rows<kHq, RPL>(Fy, Fn, lane, y);
#pragma unroll
                for (int h = 0; h < RPL; ++h) m[h] = Py[h] & Fn[h] & ~Wn[h] & vrow2[h];
                if (any(m)) {
                    moved = true;
                    prev_rows<kHq, RPL>(m, mp, lane, y);
#pragma unroll
                    for (int h = 0; h < RPL; ++h) {
                        Py[h] = (Py[h] & ~m[h]) | mp[h];
                        Fy[h] &= ~mp[h];
                    }
                }
                next_rows<kHq, RPL>(Py, Pn, lane, y);
#pragma unroll
                for (int h = 0; h < RPL; ++h) m[h] = Fy[h] & ~Wy[h] & Pn[h] & vrow2[h];
                if (any(m)) {
                    moved = true;
                    prev_rows<kHq, RPL>(m, mp, lane, y);
#pragma unroll
                    for (int h = 0; h < RPL; ++h) {
                        Py[h] = (Py[h] & ~mp[h]) | m[h];
                        Fy[h] &= ~m[h];
                    }
                }
            }
            if (g == 0) {
#pragma unroll
                for (int h = 0; h < RPL; ++h) {
                    if (rw[h]) F[yr[h]] = Fy[h];
                    if (rw[h] && moved) P2[yr[h]] = Py[h];
                }
            }
            lds_order();
            const uint32_t none[RPL] = {};
            uint64_t applied = 0ull;              // rules that applied in this step
            int w = 0;                            // loaded rules before w are done
            while (w < nl) {
                uint32_t cand = probe(w);
                int stop = -1;                    // the rule that applied
                while (cand && stop < 0) {
                    int c[kG];
#pragma unroll
                    for (int q = 0; q < kG; ++q) {
                        c[q] = cand ? kMoveRules + w + __builtin_ctz(cand) : Rt;
                        if (cand) cand &= cand - 1u;
                    }
                    uint32_t f = finish(c[0], c[1], c[2], c[3]);
                    for (; f && stop < 0; f &= f - 1u) {
                        const int q = __builtin_ctz(f);
                        const int r = q == 0 ? c[0] : q == 1 ? c[1] : q == 2 ? c[2] : c[3];
                        if (!CTL || control(r, applied, nbase + uint64_t(k))) stop = r;
                    }
                }
                if (stop < 0) {
                    w += 2 * kG;
                    continue;
                }
                applied |= 1ull << stop;
                cast(stop);
                write(uniform(PT[stop * kProbeWords + 7]), 1ull << stop, none, none);
                w = stop - kMoveRules + 1;
            }
        } else {
            next_rows<kHq, RPL>(Fy, Fn, lane, y);
            // the four moves (rules 0..3: right, left, down, up) and their votes on the player
            // plane; group 0 stores their match rows for an exact recount
            uint32_t m0[RPL], m1[RPL], m2[RPL], m3[RPL], m2p[RPL], m3p[RPL];
            uint32_t mplus[RPL], mminus[RPL], pnew[RPL];
#pragma unroll
            for (int h = 0; h < RPL; ++h) {
                m0[h] = Py[h] & (Fy[h] >> 1) & ~(Wy[h] >> 1) & cm1;
                m1[h] = Fy[h] & ~Wy[h] & (Py[h] >> 1) & cm1;
                m2[h] = Py[h] & Fn[h] & ~Wn[h] & vrow2[h];
                m3[h] = Fy[h] & ~Wy[h] & Pn[h] & vrow2[h];
            }
            prev_rows<kHq, RPL>(m2, m2p, lane, y);
            prev_rows<kHq, RPL>(m3, m3p, lane, y);
            uint32_t both = 0u;
#pragma unroll
            for (int h = 0; h < RPL; ++h) {
                mplus[h] = (m0[h] << 1) | m1[h] | m2p[h] | m3[h];
                mminus[h] = m0[h] | (m1[h] << 1) | m2[h] | m3p[h];
                pnew[h] = (Py[h] | mplus[h]) & ~mminus[h];
                both |= mplus[h] & mminus[h];
            }
            if (g == 0) {
#pragma unroll
                for (int h = 0; h < RPL; ++h) {
                    if (rw[h]) F[yr[h]] = Fy[h];
                    M[0 * MS + PAD + yr[h]] = m0[h];
                    M[1 * MS + PAD + yr[h]] = m1[h];
                    M[2 * MS + PAD + yr[h]] = m2[h];
                    M[3 * MS + PAD + yr[h]] = m3[h];
                }
            }
            lds_order();
            // every loaded rule's matches on this map
            uint64_t cand = 0ull, fired = 0ull;
            for (int w = 0; w < nl; w += 2 * kG) cand |= uint64_t(probe(w)) << (kMoveRules + w);
            while (cand) {
                int c[kG];
#pragma unroll
                for (int q = 0; q < kG; ++q) {
                    c[q] = cand ? __builtin_ctzll(cand) : Rt;
                    if (cand) cand &= cand - 1ull;
                }
                const uint32_t f = finish(c[0], c[1], c[2], c[3]);
#pragma unroll
                for (int q = 0; q < kG; ++q) fired |= ((f >> q) & 1u) ? 1ull << c[q] : 0ull;
            }
            if constexpr (CTL) {
                uint64_t applied = 0ull;
                for (uint64_t fr = fired; fr; fr &= fr - 1ull) {
                    const int r = __builtin_ctzll(fr);
                    if (control(r, applied, nbase + uint64_t(k))) applied |= 1ull << r;
                }
                fired = applied;
            }
            for (uint64_t fr = fired; fr; fr &= fr - 1ull) cast(__builtin_ctzll(fr));
            // the player plane by the moves' votes alone, counted exactly where some cell got
            // votes of both signs (then the channel is recounted with the loaded rules' votes, of
            // which there may be none)
            uint32_t which = lvoted;
            if (!((which >> kChPlayer) & 1u)) {
                if (__builtin_amdgcn_ballot_w64(both != 0u)) {
                    which |= 1u << kChPlayer;
                } else if (g == 0) {
#pragma unroll
                    for (int h = 0; h < RPL; ++h)
                        if (rw[h]) P2[yr[h]] = pnew[h];
                }
            }
            lds_order();
            write(which, fired, mplus, mminus);
            lvoted = which;
#pragma unroll
            for (int h = 0; h < RPL; ++h) Py[h] = pnew[h];
        }

        // reward: the sum over group 0's lanes
        if (__builtin_amdgcn_ballot_w64(rsum != 0))
            rsum = __builtin_amdgcn_readlane(group_prefix(rsum), kHq - 1);
        // the lane's player and wall rows, read again when a loaded rule voted on either plane
        if (lvoted & ((1u << kChPlayer) | (1u << kChWall))) {
#pragma unroll
            for (int h = 0; h < RPL; ++h) {
                Py[h] = rw[h] ? P2[yr[h]] : 0u;
                Wy[h] = rw[h] ? P[kChWall * PR + yr[h]] : 0u;
            }
        }
        const bool anyp = __builtin_amdgcn_ballot_w64(any_row<RPL>(Py)) != 0ull;
        t_env += 1;
        const bool d = !anyp || (a.L > 0 && t_env == a.L);
        if (d) {                                  // back to the initial rows
            t_env = 0;
#pragma unroll
            for (int h = 0; h < RPL; ++h) {
                if (rw[h]) {
#pragma unroll 1
                    for (int c = g; c < C; c += kG) P[c * PR + yr[h]] = I0[c * HR + yr[h]];
                }
                Py[h] = rw[h] ? I0[kChPlayer * HR + yr[h]] : 0u;
                Wy[h] = rw[h] ? I0[kChWall * HR + yr[h]] : 0u;
            }
        }
        lds_order();
        if (lane == kb) {
            rbuf = float(rsum);
            dbuf = d ? 1u : 0u;
        }
        if (kb == 63 || k == a.k - 1) {
            const int k0 = k - kb;
            if (lane <= kb) {
                a.rewards[size_t(k0 + lane) * a.B + b] = rbuf;
                a.done[size_t(k0 + lane) * a.B + b] = uint8_t(dbuf);
            }
        }
    }

    {
        const int rcs = 64 / H, rcl = lane / H, rrow = lane - rcl * H;
        if (rcl < rcs) {
            for (int c = rcl; c < C; c += rcs) {
                const size_t at = (size_t(c) * a.B + b) * H + rrow;
                if (a.row_bytes == 2) static_cast<uint16_t *>(a.state)[at] = uint16_t(P[c * PR + rrow]);
                else static_cast<uint32_t *>(a.state)[at] = P[c * PR + rrow];
            }
        }
    }
    if (lane == 0) {
        a.t[b] = t_env;
        a.nctr[b] = nbase + uint64_t(a.k);
        if (a.cost) {
            const uint64_t c = (__builtin_amdgcn_s_memtime() - t_start) >> 8;
            a.cost[b] = uint32_t(c < 0xFFFFFFFFull ? c : 0xFFFFFFFFull);
        }
    }
}

int solo_rows(int H) { return H <= 16 ? 16 : 32; }

size_t solo_base_bytes(int H, int W, int C, int rules_per_set, int max_pat_h, bool sequential,
                       bool control, bool random) {
    const int HR = solo_rows(H), PR = group_plane_words(HR, max_pat_h), NC = sequential ? C + 1 : C;
    return sizeof(uint32_t) *
           (size_t(C + 1) * PR + size_t(rules_per_set) * PR + size_t(2 * NC + C) * HR +
            size_t(rules_per_set + 1) * kProbeWords + size_t(NC) * (rules_per_set + 2) +
            (control ? size_t(3) * rules_per_set : 0) +
            (control && random ? size_t(H) * key_stride(W) : 0));
}

template <int RPL, int NJ, bool SEQ, bool CTL>
void launch_prog(const StepArgs &a, size_t lds, bool prog_lds, hipStream_t s) {
    if (prog_lds)
        hipLaunchKernelGGL((solo_step<RPL, NJ, SEQ, CTL, true>), dim3(a.B), dim3(64), lds, s, a);
    else
        hipLaunchKernelGGL((solo_step<RPL, NJ, SEQ, CTL, false>), dim3(a.B), dim3(64), lds, s, a);
}
template <int RPL, int NJ>
void launch_mode(const StepArgs &a, size_t lds, bool prog_lds, hipStream_t s) {
    if (a.sequential && a.ctl.active) launch_prog<RPL, NJ, true, true>(a, lds, prog_lds, s);
    else if (a.sequential) launch_prog<RPL, NJ, true, false>(a, lds, prog_lds, s);
    else launch_prog<RPL, NJ, false, true>(a, lds, prog_lds, s);
}

}  // namespace

bool solo_eligible(int H, int W, int C, int rules_per_set, int max_pat_h, int max_pat_w,
                   bool sequential, bool control, bool random) {
    if (H > 32 || W > 32 || (!sequential && !control)) return false;
    // rule masks are 64-bit; a recount's 8-bit counters hold the votes one cell-channel can get
    // (each from a distinct rule and pattern cell; in sequential order of one rule); the probe
    // table's offsets are 16-bit and merged entries address plane rows in 12 bits
    const long cells = long(max_pat_h) * max_pat_w;
    if (rules_per_set > 64 || (sequential ? 1 : rules_per_set) * cells > 254) return false;
    if (long(rules_per_set) * (C + 1) * cells > 0xFFFF) return false;
    return (C + 1) * group_plane_words(solo_rows(H), max_pat_h) <= kMaxEntryOffset + 1 &&
           solo_base_bytes(H, W, C, rules_per_set, max_pat_h, sequential, control, random) <=
               size_t(kLdsBudget);
}

hipError_t launch_solo_step(const StepArgs &a, hipStream_t s) {
    const size_t base = solo_base_bytes(a.H, a.W, a.C, a.prog.rules_per_set, a.max_pat_h,
                                        a.sequential != 0, a.ctl.active != 0, a.ctl.random != 0);
    const size_t prog = sizeof(uint32_t) * (size_t(a.prog.rules_per_set) * kHdrWords +
                                            a.prog.gmatch_stride + a.prog.rvote_stride +
                                            2 * (a.C + 1) + a.prog.vote_stride);
    // the program goes to LDS for launches of 16 steps or more, when it fits and leaves room
    // for as many waves per CU (160 KiB of LDS) as the batch can use, up to 8 (2 per SIMD)
    const size_t need = size_t(std::min(8, (a.B + 255) / 256));
    const size_t budget = std::min(size_t(kLdsBudget), size_t(160) * 1024 / need);
    const bool prog_lds = a.k >= kProgLdsSteps && base + prog <= budget;
    const size_t lds = base + (prog_lds ? prog : 0);
    const bool narrow = a.max_pat_w <= 3;
    if (solo_rows(a.H) == 16) {
        if (narrow) launch_mode<1, 3>(a, lds, prog_lds, s);
        else launch_mode<1, 8>(a, lds, prog_lds, s);
    } else {
        if (narrow) launch_mode<2, 3>(a, lds, prog_lds, s);
        else launch_mode<2, 8>(a, lds, prog_lds, s);
    }
    return hipGetLastError();
}

}  // namespace av
