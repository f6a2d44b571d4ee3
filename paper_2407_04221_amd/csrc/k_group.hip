// group engine: one environment per wave, its rules dealt to groups of lanes.
//
// Lane y of each of the wave's four groups of 16 lanes owns map row y (a 32-bit word, bit x =
// column x) and, on maps of 17 to 32 rows, row y + 16 too (HR = 16 or 32 rows).  One workgroup is
// one wave, so a step needs no barrier: the wave's LDS operations take effect in the order it
// issues them.  The wave engine (k_wave.hip) runs the same kernel in its other modes: sequential
// rule order (SEQ) and rule application control (CTL).
//
// What bounds it: with four waves per SIMD the VALU work of testing pattern entries, with one wave
// per SIMD the chain of dependent LDS round trips of a step, and a launch lasts as long as its
// slowest environment.  So a step tests no more than it has to:
//   - only anchors whose pattern can reach a cell that changed since the rule was last tested
//     are tested again; a rule's other matches stand (M holds them from step to step).  Most
//     steps move a player and its force, a few rows of the map, so
//   - the rows to test are a window: eight lanes per rule, so eight rules at once, one row a lane
//     when the window has at most 8 rows, else every row of the map (two or four a lane: what an
//     entry's test costs beside its rows is shared by them);
//   - a rule is probed with four merged entries (one LDS read tests every specified column of a
//     pattern row), or eight, those that accept the fewest cells first, and only rules that still
//     hold an anchor are finished, dealt to the octets as they come up.
// Within a launch only: a launch's first step, and a step after a reset, tests every anchor.
//
// Measured (MI355X, one rule set per environment, us per step in long launches, against the form
// that tested every anchor of every step with 16 lanes per rule and OR-ed votes before counting
// them): 1024 maps of 16 x 16, 8 rules, random / planted on the first map / dense 0.83 / 2.34 / 24.4
// -> 0.78 / 1.66 / 8.9; 4096 of 32 x 32, 16 rules 7.3 / 14.1 / 67.6 -> 6.2 / 11.7 / 35.3; one step of
// those with its observation 41.7 -> 33.0.  Against k_wave.hip's several waves per environment: at
// launch_wave_step, which takes this kernel for sequential order and control.  A one-wave kernel of
// their own, which tested every anchor, was ahead of these modes with few rules that seldom fire
// (50 sequential steps of 777 maps of 23 x 19, 7 rules, random / planted / dense 327 / 545 / 1940 us
// against 362 / 656 / 1406 here) and behind with more (1024 of 32 x 32, 16 rules 113 / 406 / 5662
// against 81 / 282 / 5404; every rule capped at a random site and inhibiting the next 1813 against
// 1061).
//
// LDS (32-bit rows):
//   P    [C+1][PR]     the map and the force plane (channel C); PR = HR + PAD rounded up to 4
//                      rows (PAD: the largest pattern's rows - 1, at least the 1 of the two-row
//                      built-in moves), so a lane reads row y + i of any pattern entry without a
//                      bounds test (rows H .. PR - 1 stay zero)
//   M    [R+5][PR]     match planes, row y at PAD + y: the zero rows above let a vote read
//                      match row y - i without a test (plane R + 4: zeros, read by votes past the
//                      end of a list); MV [R+4][PR] the same after control (CTL; else M)
//   DR   [HR]          anchors to test, Q [R][HR] a window's matches
//   the head of the set's table:
//   PT   [R+5][12]     per rule its first four merged entries, anchor rows and columns, place of
//                      its entries, reward, voted channels, its next four entries (row R + 4:
//                      zeros, no anchors)
//   RS   [NC][R+4]     per channel and rule, the place and number of the rule's votes in the
//                      channel's list and how many are minus votes (NC: C, or C + 1 in sequential
//                      order, where later rules read the force plane)
//   CT   [R+4][3]      control: the rule's cap and its inhibitors' mask
//   KEY  [H][W|1]      random site order: the step's index channel (32 words of slack)
//   the rest of the table, in LDS as far as it fits (see the launcher): GM the merged entries,
//                      CV the vote lists by channel
//
// Per step (paper Sec. 2.1, Sec. 2.1.1, Sec. 2.2.1), parallel rule order:
//   force  F[y] = the player row moved one cell toward the action (group 0 writes it);
//   moves  right P & (F >> 1) & ~(W >> 1), left F & ~W & (P >> 1), down P & F' & ~W', up
//          F & ~W & P' (primes: the next row), in registers: the player and wall rows stay in
//          registers from step to step unless a loaded rule wrote those planes;
//   match  probe and finish over the window; a rule's new match plane is its old one outside the
//          tested anchors and the window's matches inside;
//   control (CTL) the fired rules in index order: matches whose patch overlaps an applied match of
//          an inhibiting rule are dropped, then at most `cap` kept, those first in row-major order
//          or with the largest keys;
//   write  the channels the fired rules voted on, eight at a time, one per octet: one bit-sliced
//          counter over every fired rule's votes on the channel: new = (old + #plus > #minus);
//   end    done when no player bit is left or the counter reaches L; reward = sum over fired
//          rules of reward * popcount; done environments return to their initial rows.
// Sequential rule order: the moves one after another in registers; then every rule is matched and,
// in order, each rule that matches applies (after its control) and writes, and the rules behind it
// are matched again where its changes reach.  The result is that of applying every rule in turn,
// at one round per rule that applies instead of one per rule.
//
// A cap in random order: every lane takes eight cells of each of its rows (cells 8 g + i of group
// g) and holds their keys, 0 where the rule does not match (a key is never 0: its low bits are the
// rank 4095 - pos, and pos is at most 1023), so the wave holds every match's key in registers.  Up
// to four matches are kept by as many maxima over the wave; more by the threshold T with exactly
// `cap` keys at or above it, found bit by bit from the top (one ballot per held key and bit; keys
// never tie).
#include <algorithm>
#include <cstring>
#include <type_traits>

#include "av_internal.h"
#include "philox.h"

#define AV_INLINE __attribute__((always_inline))

namespace av {
namespace {

constexpr int kHq = 16;                 // lanes of a group
constexpr int kG = 4;                   // groups of a wave
constexpr int kProbeEntries = 4;        // merged entries of a rule tested in one round
constexpr int kProbeWords = 12;         // probe table row: entries 0-3, anchor word, match
                                        // offset | count << 16, reward, voted channels, entries
                                        // 4-7
// Input entries merged per plane row: o | jb << 12 | zero << 16 | one << 24 tests row o + y of the
// planes (o = c * PR + i: pattern row i of plane c) at the pattern columns 8 jb + j, j < 8: a cell
// of a column in `zero` must be 0, of a column in `one` must be 1.  kPassEntry tests no column (it
// passes everywhere).
constexpr uint32_t kPassEntry = 0u;
constexpr int kMaxEntryOffset = 4095;
constexpr uint32_t kMoreEntries = 1u << 16;   // of an anchor word: more entries than the probe's eight
// Votes of a channel's list: byte offset of the rule's match row y - i from that of row y of rule
// 0 (16 bits) | j << 16 | bit 31 for a minus vote.
constexpr uint32_t kMinusVote = 0x80000000u;
constexpr size_t kCuLds = 160 * 1024;   // LDS of a compute unit
constexpr int kMaxChan = 32;            // channels with a vote list
constexpr int kKeyCells = 8;            // cells of a row one lane holds keys for
constexpr int kShortLaunch = 16;        // launches of fewer steps read the lists from memory

// Words per plane row block: HR rows plus the pattern rows hanging below the last one,
// rounded up to 4 (16-byte aligned table after the planes).
__host__ __device__ constexpr int group_plane_words(int rows, int pat_rows) {
    return (rows + pat_rows - 1 + 3) & ~3;
}
// Rows of the tallest pattern, the built-in moves (two rows) among the patterns: with loaded
// patterns of one row, too, the moves' votes read the match row above a cell's.  The host lays out
// the planes by it and gives it to the kernel as max_pat_h.
constexpr int pattern_rows(int max_pat_h) { return max_pat_h > 2 ? max_pat_h : 2; }
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
__host__ __device__ constexpr int key_stride(int W) { return W | 1; }
// Words of a table's head (PT and RS), rounded up to 4.
__host__ __device__ constexpr int group_head_words(int rules_per_set, int lists) {
    return ((rules_per_set + 1) * kProbeWords + lists * rules_per_set + 3) & ~3;
}
// Map rows a lane group covers: its 16 lanes hold one row each, or two on maps of 17 to 32 rows.
constexpr int group_rows(int H) { return H <= 16 ? 16 : 32; }

__device__ inline uint32_t low_mask(int bits) { return bits >= 32 ? ~0u : ((1u << bits) - 1u); }
__device__ inline uint32_t uniform(uint32_t v) {
    return uint32_t(__builtin_amdgcn_readfirstlane(int(v)));
}
template <int CTRL>
__device__ inline uint32_t dpp(uint32_t v) {
    return uint32_t(__builtin_amdgcn_update_dpp(0, int(v), CTRL, 0xF, 0xF, true));
}

// Orders the wave's LDS writes before its later LDS reads for the compiler (the hardware keeps
// a wave's LDS operations in order, and no instruction comes of it).
__device__ inline void lds_order() { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); }

// Copy n words (a multiple of 4, both 16-byte aligned) from global memory to LDS, four loads of a
// lane in flight before its writes.
__device__ inline void copy_to_lds(uint32_t *dst, const uint32_t *src, int n, int lane) {
    u32x4 *const d = reinterpret_cast<u32x4 *>(dst);
    const u32x4 *const s = reinterpret_cast<const u32x4 *>(src);
    const int m = n >> 2;
    for (int w0 = lane; w0 < m; w0 += 4 * 64) {
        u32x4 v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int w = w0 + 64 * u;
            v[u] = w < m ? s[w] : u32x4{0u, 0u, 0u, 0u};
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int w = w0 + 64 * u;
            if (w < m) d[w] = v[u];
        }
    }
}

// The groups of eight lanes with a lane in `bal`: bit w for lanes 8 w .. 8 w + 7.
__device__ inline uint32_t octets_of(unsigned long long bal) {
    bal |= bal >> 4;
    bal |= bal >> 2;
    bal |= bal >> 1;
    bal &= 0x0101010101010101ull;                 // bit 0 of every byte, then side by side
    return uint32_t((bal * 0x0102040810204080ull) >> 56);
}

// Inclusive prefix sum over the 16 lanes of a group.
__device__ inline uint32_t group_prefix(uint32_t v) {
    v += dpp<0x111>(v);                           // row_shr by 1, 2, 4, 8
    v += dpp<0x112>(v);
    v += dpp<0x114>(v);
    v += dpp<0x118>(v);
    return v;
}
// Sum over eight lanes, or the 16 of a group, in every lane.
__device__ inline uint32_t octet_sum(uint32_t v) {
    v += dpp<0x141>(v);                           // row_half_mirror: lanes 7 - i of 8
    v += dpp<0xB1>(v);                            // lanes i ^ 1, i ^ 2
    v += dpp<0x4E>(v);
    return v;
}
__device__ inline uint32_t group_sum(uint32_t v) {
    v = octet_sum(v);
    return v + dpp<0x128>(v);                     // row_ror by 8
}
// Maximum over the wave (uniform).
__device__ inline uint32_t wave_max(uint32_t v) {
    v = max(v, dpp<0x128>(v));
    v = max(v, dpp<0x124>(v));
    v = max(v, dpp<0x122>(v));
    v = max(v, dpp<0x121>(v));
    uint32_t m = 0u;
#pragma unroll
    for (int gg = 0; gg < kG; ++gg)
        m = max(m, uint32_t(__builtin_amdgcn_readlane(int(v), kHq * gg)));
    return m;
}
// OR over the four groups (lanes y, y + 16, y + 32, y + 48).
__device__ inline uint32_t groups_or(uint32_t v) {
    const auto p = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    v = p[0] | p[1];
    const auto q = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    return q[0] | q[1];
}

// Rows y + 1 (next) and y - 1 (prev) of the rows a lane holds, 0 past the group's ends, RPL
// of them (2: on maps of 17 to 32 rows a lane of a 16-lane group holds rows y and y + 16):
// within each 16-row half a DPP row shift, across the halves a DPP row rotate (lane 15's next
// row is lane 0's second row, lane 0's second row's previous row is lane 15's first).
template <int RPL>
__device__ inline void next_rows(const uint32_t (&v)[RPL], uint32_t (&n)[RPL], int y) {
    if constexpr (RPL == 1) {
        n[0] = dpp<0x101>(v[0]);
    } else {
        const uint32_t s0 = dpp<0x101>(v[0]), w1 = dpp<0x12F>(v[1]), s1 = dpp<0x101>(v[1]);
        n[0] = y == kHq - 1 ? w1 : s0;
        n[1] = s1;
    }
}
template <int RPL>
__device__ inline void prev_rows(const uint32_t (&v)[RPL], uint32_t (&p)[RPL], int y) {
    if constexpr (RPL == 1) {
        p[0] = dpp<0x111>(v[0]);
    } else {
        const uint32_t s0 = dpp<0x111>(v[0]), t1 = dpp<0x111>(v[1]), w0 = dpp<0x121>(v[0]);
        p[0] = s0;
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

// Add the four one-bit planes x to the KB-bit bit-sliced counter q: carry-save adders make them a
// 3-bit number, then one ripple add.
template <int KB>
__device__ inline void count4(uint32_t (&q)[KB], uint32_t x0, uint32_t x1, uint32_t x2, uint32_t x3) {
    const uint32_t s1 = x0 ^ x1 ^ x2, c1 = (x0 & x1) | (x2 & (x0 ^ x1));   // weight 1, 2
    const uint32_t s0 = s1 ^ x3, c2 = s1 & x3;                             // weight 1, 2
    const uint32_t w2 = c1 ^ c2, w4 = c1 & c2;                             // weight 2, 4
    uint32_t k = q[0] & s0;
    q[0] ^= s0;
    const uint32_t k1 = (q[1] & w2) | (k & (q[1] ^ w2));
    q[1] = q[1] ^ w2 ^ k;
    k = (q[2] & w4) | (k1 & (q[2] ^ w4));
    q[2] = q[2] ^ w4 ^ k1;
#pragma unroll
    for (int b = 3; b < KB; ++b) {
        const uint32_t kq = q[b] & k;
        q[b] ^= k;
        k = kq;
    }
}

// RPL: map rows a lane holds: 2 on maps of 17 to 32 rows (lane y of a 16-lane group holds rows
// y and y + 16), else 1.
// NJ: columns a merged entry tests (3 when no pattern is wider, else 8).
// SEQ, CTL: sequential rule order, rule application control.
// WHERE: kLds the table's lists are copied to LDS; kEntries the merged entries are, the votes are
// read from memory; kGlobal both are.  A compile-time choice, so that the lists' reads are LDS
// reads or global loads: a pointer that may be either makes every read a flat load, which the LDS
// reads' waits then wait for as well.
// WAVES: waves per SIMD the registers must leave room for.
enum : int { kLds = 0, kEntries = 1, kGlobal = 2 };

template <int RPL, int NJ, bool SEQ, bool CTL, int WHERE, int WAVES>
__global__ void __launch_bounds__(64, WAVES) group_step(StepArgs a) {
    constexpr int HR = kHq * RPL;                 // map rows a group covers
    extern __shared__ __align__(16) uint32_t lds[];
    const int lane = int(threadIdx.x), g = lane / kHq, y = lane % kHq;
    const uint64_t t_start = __builtin_amdgcn_s_memtime();
    const int b = a.order ? a.order[blockIdx.x] : int(blockIdx.x);
    const int H = a.H, W = a.W, C = a.C, C1 = C + 1, Rt = a.prog.rules_per_set;
    const int NC = SEQ ? C1 : C;
    // pattern rows beyond a lane's row: plane rows y + i and match rows y - i, i <= PAD, are
    // read without a bounds test
    const int PAD = a.max_pat_h - 1;
    const int PR = group_plane_words(HR, a.max_pat_h), MS = PR;
    const int s = a.per_env ? b : 0;
    const int nl = Rt - kMoveRules;               // loaded rules
    // the lane's rows; past the map (rw false) their plane rows stay zero and are read freely
    // (row yr + i < PR), their anchors are masked off and they are never written
    int yr[RPL];
    bool rw[RPL];
#pragma unroll
    for (int h = 0; h < RPL; ++h) {
        yr[h] = y + kHq * h;
        rw[h] = yr[h] < H;
    }
    const uint32_t wmask = low_mask(W);
    const int head = group_head_words(Rt, NC);

    uint32_t *const P = lds;                       // [C1][PR]
    uint32_t *const M = P + C1 * PR;               // [Rt + 1][MS]
    uint32_t *const MV = CTL ? M + (Rt + 1) * MS : M;   // [Rt + 1][MS]
    uint32_t *const DR = MV + (Rt + 1) * MS;       // [HR]
    uint32_t *const Q = DR + HR;                   // [nl][HR]
    uint32_t *const PT = Q + nl * HR;              // [Rt + 1][kProbeWords]
    uint32_t *const RS = PT + (Rt + 1) * kProbeWords; // [NC][Rt]
    uint32_t *const lists = PT + head;             // merged entries, votes (WHERE)
    const int in_lds = WHERE == kLds ? a.prog.gtab_stride
                                     : head + (WHERE == kEntries ? a.prog.gentry_words : 0);
    uint32_t *const CT = PT + in_lds;              // [Rt][3] (CTL)
    uint32_t *const KEY = CT + 3 * Rt;             // [H][key_stride(W)] + 32 (random order)

    const uint32_t *const gtab = a.prog.gtab + size_t(s) * a.prog.gtab_stride;
    const uint32_t *const gm = WHERE == kGlobal ? gtab + head : lists;
    const uint32_t *const cv = (WHERE == kLds ? lists : gtab + head) + a.prog.gentry_words;

    copy_to_lds(PT, gtab, in_lds, lane);
    {
        // planes and match planes: zero; then the map's rows.  Lane l takes row l % H of channels
        // l / H, l / H + 64 / H, ..., four rows of a lane in flight
        const int rcs = 64 / H, rcl = lane / H, rrow = lane - rcl * H;
        auto zero = [&]() AV_INLINE {
            u32x4 *const z = reinterpret_cast<u32x4 *>(lds);
            const int words = int(DR - P) >> 2;
            for (int w = lane; w < words; w += 64) z[w] = u32x4{0u, 0u, 0u, 0u};
        };
        auto load_rows = [&](const auto *st) AV_INLINE {
            bool first = true;
            for (int c0 = rcl; c0 - rcl < C; c0 += 4 * rcs) {
                uint32_t sv[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int c = c0 + u * rcs;
                    sv[u] = rcl < rcs && c < C ? uint32_t(st[(size_t(c) * a.B + b) * H + rrow]) : 0u;
                }
                if (first) zero();
                first = false;
                lds_order();
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int c = c0 + u * rcs;
                    if (rcl < rcs && c < C) P[c * PR + rrow] = sv[u];
                }
            }
        };
        if (a.row_bytes == 2) load_rows(static_cast<const uint16_t *>(a.state));
        else load_rows(static_cast<const uint32_t *>(a.state));
    }
    if constexpr (CTL) {
        for (int r = lane; r < Rt; r += 64) {
            const size_t cr = size_t(s) * Rt + r;
            CT[3 * r] = uint32_t(a.ctl.limit[cr]);
            CT[3 * r + 1] = a.ctl.inhibit[cr * a.ctl.words];
            CT[3 * r + 2] = a.ctl.words > 1 ? a.ctl.inhibit[cr * a.ctl.words + 1] : 0u;
        }
    }
    int t_env = a.t[b];
    const uint64_t nbase = a.nctr[b];
    __syncthreads();   // (one wave: orders the set-up's LDS writes before the step's reads)

    // The window: eight lanes per rule (or channel), this lane in octet wo at place wl, at rows
    // wr + 8 h (h < RP: one row, or FULL when the window is every row of the map).
    constexpr int FULL = HR / 8;
    // with four waves per SIMD (128 registers) probe rows stay in LDS and, with two rows a lane, a
    // write of every row is made in two halves, or registers would spill
    constexpr bool HELD = WAVES < 4, HALVES = RPL == 2 && WAVES == 4;
    const int wo = lane >> 3, wl = lane & 7;
    int wr = wl, r0 = 0;                          // r0: the window's first row
    // four merged entries at the window's rows: the anchors m they leave.  A column's bits of an
    // entry sign-extended are masks; what a column rejects is gathered unshifted over the four
    // entries and moved right by the column's offset once (the cells that the shift would bring in
    // from past the map's edge are no anchors)
    auto entries4 = [&](const u32x4 &e4, auto &m) AV_INLINE {
        constexpr int RP = sizeof(m) / sizeof(m[0]);
        const uint32_t e[4] = {e4.x, e4.y, e4.z, e4.w};
        uint32_t v[4][RP], bad[RP];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
#pragma unroll
            for (int h = 0; h < RP; ++h) v[u][h] = P[int(e[u] & uint32_t(kMaxEntryOffset)) + wr + 8 * h];
        }
        if constexpr (NJ > 3) {
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int h = 0; h < RP; ++h) v[u][h] >>= (e[u] >> 9) & 24u;
        }
#pragma unroll
        for (int h = 0; h < RP; ++h) bad[h] = 0u;
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            uint32_t o[RP];
#pragma unroll
            for (int h = 0; h < RP; ++h) o[h] = 0u;
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const uint32_t zero = uint32_t(int32_t(e[u] << (15 - j)) >> 31);
                const uint32_t one = uint32_t(int32_t(e[u] << (7 - j)) >> 31);
#pragma unroll
                for (int h = 0; h < RP; ++h) o[h] |= (v[u][h] & zero) | (~v[u][h] & one);
            }
#pragma unroll
            for (int h = 0; h < RP; ++h) bad[h] |= o[h] >> j;
        }
#pragma unroll
        for (int h = 0; h < RP; ++h) m[h] &= ~bad[h];
    };
    // table row of loaded rule i (none: row Rt, which has no anchors)
    auto row_of = [&](int i) AV_INLINE { return PT + (i < nl ? kMoveRules + i : Rt) * kProbeWords; };
    // the probe entries and anchor words of loaded rules wo and wo + 8, held for the launch (if HELD)
    auto held = [&](int i, u32x4 &e, uint32_t &v) AV_INLINE {
        const uint32_t *const row = row_of(i);
        e = *reinterpret_cast<const u32x4 *>(row);
        v = row[4];
    };
    u32x4 ha0, ha1;
    uint32_t hav0, hav1;
    if constexpr (HELD) {
        held(wo, ha0, hav0);
        held(8 + wo, ha1, hav1);
    }
    // probe of loaded rules w .. w + 7 (or w + 15) over the window, rule w + wo (and w + 8 + wo) by
    // this lane's octet, among the anchors t: their first four entries and, where some rule keeps
    // an anchor, the next four; where one still does, the window's rows so far go to Q: rules
    // without more entries match there (hit), the others are returned (loaded rules).  (On crowded
    // maps four entries leave most rules an anchor and eight leave few: the second four here cost
    // half of what they cost in finish, which deals the rules out again.)
    auto probe = [&](int w, bool two, const auto &t, uint64_t &hit) AV_INLINE -> uint64_t {
        constexpr int RP = sizeof(t) / sizeof(t[0]);
        uint64_t found = 0ull;
        auto start = [&](uint32_t pv, uint32_t (&m)[RP]) AV_INLINE {
#pragma unroll
            for (int h = 0; h < RP; ++h)
                m[h] = wr + 8 * h < int((pv >> 8) & 255u) ? t[h] & (~0u >> (pv & 255u)) : 0u;
        };
        auto keep = [&](int i, uint32_t pv, const uint32_t (&m)[RP], int at) AV_INLINE {
            const unsigned long long bal = __builtin_amdgcn_ballot_w64(any_row<RP>(m));
            if (!bal) return;
            if (i < nl) {
#pragma unroll
                for (int h = 0; h < RP; ++h) Q[i * HR + wl + 8 * h] = m[h];
            }
            const unsigned long long more = bal & __builtin_amdgcn_ballot_w64((pv & kMoreEntries) != 0u);
            hit |= uint64_t(octets_of(bal & ~more)) << at;
            found |= uint64_t(octets_of(more)) << at;
        };
        const int i0 = w + wo, i1 = w + 8 + wo;
        uint32_t m0[RP], m1[RP];
        u32x4 e0, e1;
        uint32_t v0, v1;
        if (HELD && w == 0) {
            e0 = ha0;
            v0 = hav0;
            e1 = ha1;
            v1 = hav1;
            // (opaque: the columns' masks, formed ahead of the step loop, would take the registers)
            asm volatile("" : "+v"(e0), "+v"(e1));
        } else {
            held(i0, e0, v0);
            held(i1, e1, v1);
        }
        start(v0, m0);
        entries4(e0, m0);
        if (two) {
            start(v1, m1);
            entries4(e1, m1);
            if (!__builtin_amdgcn_ballot_w64(any_row<RP>(m0) || any_row<RP>(m1))) return 0ull;
            e0 = *reinterpret_cast<const u32x4 *>(row_of(i0) + 8);
            e1 = *reinterpret_cast<const u32x4 *>(row_of(i1) + 8);
            entries4(e0, m0);
            entries4(e1, m1);
            keep(i0, v0, m0, w);
            keep(i1, v1, m1, w + 8);
        } else {
            if (!__builtin_amdgcn_ballot_w64(any_row<RP>(m0))) return 0ull;
            entries4(*reinterpret_cast<const u32x4 *>(row_of(i0) + 8), m0);
            keep(i0, v0, m0, w);
        }
        lds_order();
        return found;
    };
    // The entries from the ninth on of the first eight loaded rules of `cand`, one per octet, over
    // the window; their matches go to Q.  Takes them out of cand; returns those
    // that match somewhere.
    auto finish = [&](uint64_t &cand, auto rp) AV_INLINE -> uint64_t {
        constexpr int RP = decltype(rp)::value;
        int i = nl;                               // the octet's rule
        uint64_t left = cand;
        for (int q = 0; q < 8 && left; ++q, left &= left - 1ull)
            i = wo == q ? __builtin_ctzll(left) : i;
        const uint64_t taken = cand & ~left;
        cand = left;
        const uint32_t meta = row_of(i)[5];
        uint32_t m[RP];
#pragma unroll
        for (int h = 0; h < RP; ++h) m[h] = i < nl ? Q[(i < nl ? i : 0) * HR + wl + 8 * h] : 0u;
        const int off = int(meta & 0xFFFFu), cnt = int(meta >> 16);
        auto four = [&](int pos) AV_INLINE -> u32x4 {   // (reads stay inside the rule's entries)
            const bool on = pos < cnt;
            u32x4 x;
            x.x = on ? gm[off + pos] : kPassEntry;
            x.y = on ? gm[off + min(pos + 1, cnt - 1)] : kPassEntry;
            x.z = on ? gm[off + min(pos + 2, cnt - 1)] : kPassEntry;
            x.w = on ? gm[off + min(pos + 3, cnt - 1)] : kPassEntry;
            return x;
        };
        u32x4 x = four(2 * kProbeEntries);
        for (int pos = 2 * kProbeEntries; __builtin_amdgcn_ballot_w64(any_row<RP>(m) && pos < cnt);) {
            pos += kProbeEntries;
            const u32x4 nx = four(pos);
            entries4(x, m);
            x = nx;
        }
        if (i < nl) {
#pragma unroll
            for (int h = 0; h < RP; ++h) Q[i * HR + wl + 8 * h] = m[h];
        }
        const uint32_t f = octets_of(__builtin_amdgcn_ballot_w64(any_row<RP>(m)));
        lds_order();
        // the rules of the octets in f: the q-th of `taken` for bit q
        uint64_t hit = 0ull;
        int q = 0;
        for (uint64_t tk = taken; tk; tk &= tk - 1ull, ++q)
            hit |= ((f >> q) & 1u) ? tk & (0ull - tk) : 0ull;
        return hit;
    };

    // Cells that changed since the rules were last tested (the lane's rows), and the anchors whose
    // pattern can reach one (Dd): pw - 1 columns to the left and ph - 1 rows up.  Returns the rows
    // that hold such an anchor.
    uint32_t Dd[RPL];
    auto spread = [&](const uint32_t (&D)[RPL]) AV_INLINE -> uint32_t {
        uint32_t t[RPL];
#pragma unroll
        for (int h = 0; h < RPL; ++h) {
            if constexpr (NJ == 3) {
                t[h] = D[h] | (D[h] >> 1) | (D[h] >> 2);   // (a pattern is at most 3 wide)
            } else {
                t[h] = D[h];
                for (int j = 1; j < a.max_pat_w; ++j) t[h] |= D[h] >> j;
            }
            Dd[h] = t[h];
        }
        for (int i = 1; i <= PAD; ++i) {
            next_rows<RPL>(t, t, y);
#pragma unroll
            for (int h = 0; h < RPL; ++h) Dd[h] |= t[h];
        }
        uint32_t rows = 0u;
#pragma unroll
        for (int h = 0; h < RPL; ++h) {
            rows |= uint32_t(__builtin_amdgcn_ballot_w64(Dd[h] != 0u) & 0xFFFFull) << (kHq * h);
            if (g == 0) DR[yr[h]] = Dd[h];
        }
        lds_order();
        return rows;
    };
    // the window for the anchors' rows; true: every row of the map (FULL rows a lane)
    auto window = [&](uint32_t rows) AV_INLINE -> bool {
        const int lo = __builtin_ctz(rows), hi = 31 - __builtin_clz(rows);
        const bool all = hi - lo >= 8;
        r0 = all ? 0 : min(lo, HR - 8);
        wr = r0 + wl;
        return all;
    };
    // rule r's new match plane: its matches so far outside the tested anchors (if `had`), the
    // window's (if `hit`) inside; false when it is empty
    auto settle = [&](int r, bool had, bool hit) AV_INLINE -> bool {
        uint32_t m[RPL];
#pragma unroll
        for (int h = 0; h < RPL; ++h) {
            m[h] = had ? M[r * MS + PAD + yr[h]] & ~Dd[h] : 0u;
            const int l = yr[h] - r0;
            // (the window of every row: r0 = 0 and HR rows)
            if (hit && l >= 0 && l < HR) {
                const uint32_t q = Q[(r - kMoveRules) * HR + l];
                m[h] |= q & Dd[h];
            }
            M[r * MS + PAD + yr[h]] = m[h];
        }
        lds_order();
        return __builtin_amdgcn_ballot_w64(any_row<RPL>(m)) != 0ull;
    };

    uint64_t live = 0ull;                         // the rules with matches in M
    // Matches of loaded rules w and on against the map as it is, D holding at least the cells that
    // changed since each of them was last matched: M and live.
    auto match = [&](const uint32_t (&D)[RPL], int w) AV_INLINE {
        const uint32_t rows = spread(D);
        if (!rows) return;
        uint64_t hit = 0ull;
        auto scan = [&](const auto &t) AV_INLINE {
            constexpr int RP = sizeof(t) / sizeof(t[0]);
            uint64_t cand = 0ull;
            for (int v = w; v < nl; v += 16) cand |= probe(v, v + 8 < nl, t, hit);
            while (cand) hit |= finish(cand, std::integral_constant<int, RP>{});
        };
        if (window(rows)) {
            uint32_t t[FULL];
#pragma unroll
            for (int h = 0; h < FULL; ++h) t[h] = DR[wr + 8 * h];
            scan(t);
        } else {
            const uint32_t t[1] = {DR[wr]};
            scan(t);
        }
        hit <<= kMoveRules;
        for (uint64_t z = hit | (live >> (kMoveRules + w) << (kMoveRules + w)); z; z &= z - 1ull) {
            const uint64_t bit = z & (0ull - z);
            live = settle(__builtin_ctzll(z), live & bit, hit & bit) ? live | bit : live & ~bit;
        }
    };

    uint32_t have_keys = 0u;                      // (random order) passes of 64 blocks in KEY
    // control of rule r, which fired on this step's map: drops inhibited matches (inhibitors among
    // `applied`) and those above the cap; false when none is left.  Every group does the same
    // work on all rows, but for the keys, which are split over the groups.  M keeps every match,
    // MV gets those that apply.
    auto control = [&](int r, uint64_t applied, uint64_t n) AV_INLINE -> bool {
        uint32_t acc[RPL];
#pragma unroll
        for (int h = 0; h < RPL; ++h) acc[h] = M[r * MS + PAD + yr[h]];
        const int lim = int(uniform(CT[3 * r]));
        const uint32_t pv = uniform(PT[r * kProbeWords + 4]);
        const int hn = H + 1 - int((pv >> 8) & 255u), hm = W - 31 + int(pv & 255u);
        uint64_t inh = (uint64_t(uniform(CT[3 * r + 1])) | (uint64_t(uniform(CT[3 * r + 2])) << 32)) & applied;
        for (; inh; inh &= inh - 1) {
            const int q = __builtin_ctzll(inh);
            const uint32_t qv = uniform(PT[q * kProbeWords + 4]);
            const int nq = H + 1 - int((qv >> 8) & 255u), mq = W - 31 + int(qv & 255u);
            // anchors of q whose patch meets an hn-row patch at the lane's rows: rows
            // y - nq + 1 .. y + hn - 1 (rows past the map are zero)
            uint32_t o[RPL], t[RPL], u[RPL];
#pragma unroll
            for (int h = 0; h < RPL; ++h) o[h] = t[h] = u[h] = MV[q * MS + PAD + yr[h]];
            for (int d = 1; d < hn; ++d) {
                next_rows<RPL>(t, t, y);
#pragma unroll
                for (int h = 0; h < RPL; ++h) o[h] |= t[h];
            }
            for (int d = 1; d < nq; ++d) {
                prev_rows<RPL>(u, u, y);
#pragma unroll
                for (int h = 0; h < RPL; ++h) o[h] |= u[h];
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
                inc[h] = int(group_prefix(uint32_t(__popc(acc[h])))) + total;
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
                    if (!have_keys) {
                        for (int p = 0; p < passes; ++p) {
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
                        have_keys = 1u;
                        lds_order();
                    }
                    uint32_t key[RPL][kKeyCells];
#pragma unroll
                    for (int h = 0; h < RPL; ++h) {
                        const uint32_t *kr = KEY + min(yr[h], H - 1) * key_stride(W) + kKeyCells * g;
                        const uint32_t f = acc[h] >> (kKeyCells * g);
#pragma unroll
                        for (int i = 0; i < kKeyCells; ++i)
                            key[h][i] = kr[i] & uint32_t(int32_t(f << (31 - i)) >> 31);
                    }
                    uint32_t T = 0u;
                    if (lim <= 4) {
                        for (int got = 0; got < lim; ++got) {   // the next largest key
                            uint32_t v = 0u;
#pragma unroll
                            for (int h = 0; h < RPL; ++h)
#pragma unroll
                                for (int i = 0; i < kKeyCells; ++i)
                                    v = max(v, got == 0 || key[h][i] < T ? key[h][i] : 0u);
                            T = wave_max(v);
                        }
                    } else {
                        for (int bit = 31; bit >= 0; --bit) {
                            const uint32_t t = T | (1u << bit);
                            int at_least = 0;
#pragma unroll
                            for (int h = 0; h < RPL; ++h)
#pragma unroll
                                for (int i = 0; i < kKeyCells; ++i)
                                    at_least += __popcll(__builtin_amdgcn_ballot_w64(key[h][i] >= t));
                            if (at_least >= lim) T = t;
                            if (at_least == lim) break;
                        }
                    }
                    // each group's kept cells, OR-ed over the groups
#pragma unroll
                    for (int h = 0; h < RPL; ++h) {
                        uint32_t keep = 0u;
#pragma unroll
                        for (int i = 0; i < kKeyCells; ++i)
                            keep |= key[h][i] >= T ? 1u << i : 0u;
                        acc[h] = groups_or(keep << (kKeyCells * g));
                    }
                }
            }
        }
#pragma unroll
        for (int h = 0; h < RPL; ++h) MV[r * MS + PAD + yr[h]] = acc[h];
        lds_order();
        return __builtin_amdgcn_ballot_w64(any_row<RPL>(acc)) != 0ull;
    };

    // New rows of the channels in `which`, eight at a time, one per octet, from the votes of the loaded
    // rules in `fu` (uniform), whose match rows OR-ed are fm: only a window of rows gets votes, and
    // with eight rows or fewer eight channels are written at once.  With `moves` the four moves'
    // votes on the player plane count too (two each, from their match rows; pn: its rows by those
    // votes alone).  A vote reads its rule's match row y - i shifted by j; a minus vote adds the
    // complement of its cells, so one counter takes old + #plus + (#minus entries - #minus votes),
    // and a cell is set, old + #plus - #minus >= 1, where it reaches 1 + #minus entries.  The
    // counters have 4, 6 or 8 bits by the most votes a channel of the round gets (a list holds at
    // most 254).  Returns in ch the cells that the votes changed.
    auto write = [&](uint32_t which, uint64_t fu, const uint32_t (&fm)[RPL], bool moves,
                     const uint32_t (&pn)[RPL], uint32_t (&ch)[RPL]) AV_INLINE {
        auto rows_of = [&](auto rp, bool half) AV_INLINE {
            constexpr int RP = decltype(rp)::value;
            const uint32_t *const mw = MV + wr;   // the lane's row of match plane 0, less PAD rows
            uint32_t cw[RP];
#pragma unroll
            for (int h = 0; h < RP; ++h) cw[h] = 0u;
            uint32_t left = which;
            while (left) {
                int c = -1;
                const uint32_t all = left;
                for (int q = 0; q < 8 && left; ++q, left &= left - 1u)
                    c = wo == q ? __builtin_ctz(left) : c;
                const bool on = c >= 0, mv = !SEQ && moves && c == kChPlayer;
                const int cc = on ? c : 0;
                const uint32_t *const rs = RS + cc * Rt;
                uint32_t old[RP];
#pragma unroll
                for (int h = 0; h < RP; ++h) old[h] = P[cc * PR + wr + 8 * h];
                lds_order();
                if (!SEQ && moves && (((all & ~left) >> kChPlayer) & 1u) && g == 0) {
#pragma unroll
                    for (int h = 0; h < RPL; ++h)     // rows without votes of loaded rules
                        if (rw[h] && (!half || (yr[h] >= r0 && yr[h] < r0 + 8 * RP)))
                            P[kChPlayer * PR + yr[h]] = pn[h];
                }
                lds_order();
                // votes and minus votes of the fired rules on c, the octet's lanes adding up theirs
                uint32_t w = rs[__builtin_ctzll(fu)], sum;
                if (fu & (fu - 1ull)) {
                    sum = 0u;
                    for (int q = 0; q < nl; q += 8) {
                        const int r = kMoveRules + q + wl;
                        const uint32_t v = rs[min(r, Rt - 1)];
                        sum += r < Rt && ((fu >> r) & 1ull) ? ((v >> 16) & 255u) | ((v >> 24) << 16) : 0u;
                    }
                    sum = octet_sum(sum);
                } else {
                    sum = ((w >> 16) & 255u) | ((w >> 24) << 16);
                }
                sum = on ? sum : 0u;
                const int total = int(sum & 0xFFFFu) + (mv ? 2 * kMoveRules : 0);
                const uint32_t need = 1u + (sum >> 16) + (mv ? kMoveRules : 0);   // 1 + #minus entries
                auto run = [&](auto kb) AV_INLINE {
                    constexpr int KB = decltype(kb)::value;
                    uint32_t cnt[RP][KB];
#pragma unroll
                    for (int h = 0; h < RP; ++h) {
#pragma unroll
                        for (int q = 1; q < KB; ++q) cnt[h][q] = 0u;
                        cnt[h][0] = old[h];
                    }
                    if (mv) {
#pragma unroll
                        for (int h = 0; h < RP; ++h) {
                            // match rows of right, left, down, up (rules 0..3) here and one above
                            const uint32_t *m = M + PAD + wr + 8 * h;
                            const uint32_t a0 = m[0], a1 = m[MS], a2 = m[2 * MS], a3 = m[3 * MS];
                            const uint32_t a2p = m[2 * MS - 1], a3p = m[3 * MS - 1];
                            count4<KB>(cnt[h], a0 << 1, a1, a2p, a3);
                            count4<KB>(cnt[h], ~a0, ~(a1 << 1), ~a2, ~a3p);
                        }
                    }
                    const uint32_t dead = uint32_t(Rt * MS) * 4u;   // the plane of zeros
                    auto add = [&](const uint32_t (&v)[4], int nv) AV_INLINE {
                        uint32_t x[RP][4];
#pragma unroll
                        for (int u = 0; u < 4; ++u) {
                            const uint32_t w = u < nv ? v[u] : dead;
                            const uint32_t *m = reinterpret_cast<const uint32_t *>(
                                reinterpret_cast<const char *>(mw) + (w & 0xFFFFu));
                            const uint32_t minus = uint32_t(int32_t(w) >> 31);
#pragma unroll
                            for (int h = 0; h < RP; ++h)
                                x[h][u] = (m[8 * h] << ((w >> 16) & 31u)) ^ minus;
                        }
#pragma unroll
                        for (int h = 0; h < RP; ++h)
                            count4<KB>(cnt[h], x[h][0], x[h][1], x[h][2], x[h][3]);
                    };
                    // the fired rules one after another (uniform), the next one's votes read with
                    // the current one's match rows; a list has slack behind its end, so four are read
                    uint64_t fr = fu;
                    uint32_t v[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) v[u] = cv[(w & 0xFFFFu) + u];
                    while (fr) {
                        fr &= fr - 1ull;
                        const uint32_t wn = rs[fr ? __builtin_ctzll(fr) : 0];
                        const int nv = on ? int((w >> 16) & 255u) : 0;
                        const uint32_t off = w & 0xFFFFu;
                        add(v, nv);
#pragma unroll 1
                        for (int e = 4; __builtin_amdgcn_ballot_w64(e < nv); e += 4) {
                            uint32_t t[4];
                            const uint32_t at = off + uint32_t(e < nv ? e : 0);
#pragma unroll
                            for (int u = 0; u < 4; ++u) t[u] = cv[at + u];
                            add(t, nv - e);
                        }
                        w = wn;
#pragma unroll
                        for (int u = 0; u < 4; ++u) v[u] = cv[(w & 0xFFFFu) + u];
                    }
#pragma unroll
                    for (int h = 0; h < RP; ++h) {
                        uint32_t gt = 0u, eq = ~0u;   // cnt >= need, bit-sliced
#pragma unroll
                        for (int q = KB - 1; q >= 0; --q) {
                            const uint32_t tb = uint32_t(int32_t(need << (31 - q)) >> 31);
                            gt |= eq & cnt[h][q] & ~tb;
                            eq &= ~(cnt[h][q] ^ tb);
                        }
                        if (on && wr + 8 * h < H) {
                            P[cc * PR + wr + 8 * h] = gt | eq;
                            cw[h] |= (gt | eq) ^ old[h];
                        }
                    }
                };
                if (!__builtin_amdgcn_ballot_w64(total > 14)) run(std::integral_constant<int, 4>{});
                else if (!__builtin_amdgcn_ballot_w64(total > 62)) run(std::integral_constant<int, 6>{});
                else run(std::integral_constant<int, 8>{});
            }
            // the changes of all channels, at the lane's own rows
#pragma unroll
            for (int h = 0; h < RP; ++h) {
                uint32_t o = cw[h];
                o = groups_or(o | dpp<0x128>(o));
                if (wo == 0) DR[wr + 8 * h] = o;
            }
        };
        // rows that get votes: from the first match row to the last one's patch's last
        uint32_t rows = 0u;
#pragma unroll
        for (int h = 0; h < RPL; ++h)
            rows |= uint32_t(__builtin_amdgcn_ballot_w64(fm[h] != 0u) & 0xFFFFull) << (kHq * h);
        const int last = min(31 - __builtin_clz(rows) + PAD, HR - 1);
        int from = 0, past = HR;                  // the rows written
        if (!window(rows | (1u << last))) {
            from = r0;
            past = r0 + 8;
            rows_of(std::integral_constant<int, 1>{}, false);
        } else if constexpr (HALVES) {
#pragma unroll 1
            for (r0 = 0; r0 < HR; r0 += HR / 2) {
                wr = r0 + wl;
                rows_of(std::integral_constant<int, FULL / 2>{}, true);
            }
        } else {
            rows_of(std::integral_constant<int, FULL>{}, false);
        }
        lds_order();
#pragma unroll
        for (int h = 0; h < RPL; ++h) ch[h] = yr[h] >= from && yr[h] < past ? DR[yr[h]] : 0u;
        lds_order();
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

    // cells that changed since the rules were last matched (in sequential order: during the step
    // before and this one) and the force rows they were matched with
    uint32_t D[RPL], Fl[RPL];
#pragma unroll
    for (int h = 0; h < RPL; ++h) {
        D[h] = rw[h] ? ~0u : 0u;
        Fl[h] = 0u;
    }

    for (int k = 0; k < a.k; ++k) {
        const int kb = k & 63;
        if (kb == 0) ablk = (k + lane < a.k) ? uint32_t(a.actions[size_t(k + lane) * a.B + b]) : 0u;
        const int act = __builtin_amdgcn_readlane(int(ablk), kb);
        if constexpr (CTL) have_keys = 0u;
        uint32_t Pn[RPL], Wn[RPL], Pp[RPL], Fy[RPL], Fn[RPL];
        next_rows<RPL>(Py, Pn, y);
        next_rows<RPL>(Wy, Wn, y);
        prev_rows<RPL>(Py, Pp, y);
#pragma unroll
        for (int h = 0; h < RPL; ++h)
            Fy[h] = act == 1 ? Pn[h] : act == 3 ? Pp[h] : act == 2 ? ((Py[h] << 1) & wmask)
                  : act == 4 ? (Py[h] >> 1) : 0u;

        uint32_t lvoted = 0u;                     // channels rewritten from LDS (uniform)
        int rsum = 0;
        // reward of rule r's match rows (a group's lanes hold them all) and the channels it votes
        // on; fm: the match rows of the rules so far
        uint32_t fm[RPL];
        auto pays = [&](int r) AV_INLINE {
            const int reward = int(uniform(PT[r * kProbeWords + 6]));
            lvoted |= uniform(PT[r * kProbeWords + 7]);
            int cells = 0;
#pragma unroll
            for (int h = 0; h < RPL; ++h) {
                const uint32_t m = MV[r * MS + PAD + yr[h]];
                fm[h] |= m;
                cells += __popc(m);
            }
            rsum += reward * cells;
        };
#pragma unroll
        for (int h = 0; h < RPL; ++h) fm[h] = 0u;

        if constexpr (SEQ) {
            // the moves one after another: right, left, down, up (each takes the player from its
            // cell to the force cell next to it and consumes the force; a cell that a player
            // leaves and another enters keeps its tile: 1 + 1 - 1)
            auto any = [&](const uint32_t (&m)[RPL]) AV_INLINE {
                return __builtin_amdgcn_ballot_w64(any_row<RPL>(m)) != 0ull;
            };
            bool moved = false;
            uint32_t F0[RPL], P0[RPL];            // the step's first force and player rows
#pragma unroll
            for (int h = 0; h < RPL; ++h) {
                Fy[h] = rw[h] ? Fy[h] : 0u;
                F0[h] = Fy[h];
                P0[h] = Py[h];
            }
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
                next_rows<RPL>(Fy, Fn, y);
#pragma unroll
                for (int h = 0; h < RPL; ++h) m[h] = Py[h] & Fn[h] & ~Wn[h] & vrow2[h];
                if (any(m)) {
                    moved = true;
                    prev_rows<RPL>(m, mp, y);
#pragma unroll
                    for (int h = 0; h < RPL; ++h) {
                        Py[h] = (Py[h] & ~m[h]) | mp[h];
                        Fy[h] &= ~mp[h];
                    }
                }
                next_rows<RPL>(Py, Pn, y);
#pragma unroll
                for (int h = 0; h < RPL; ++h) m[h] = Fy[h] & ~Wy[h] & Pn[h] & vrow2[h];
                if (any(m)) {
                    moved = true;
                    prev_rows<RPL>(m, mp, y);
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
            // what changed in this step so far: the force rows, the moves
            uint32_t Dc[RPL], ch[RPL];
#pragma unroll
            for (int h = 0; h < RPL; ++h) {
                Dc[h] = (F0[h] ^ Fl[h]) | (F0[h] ^ Fy[h]) | (P0[h] ^ Py[h]);
                D[h] |= Dc[h];
            }
            // every rule on the map after the moves; then, in order, the rules that match: each that
            // applies changes the map under the rules behind it, which are matched again where its
            // changes reach
            match(D, 0);
            uint64_t applied = 0ull;              // rules that applied in this step
            for (uint64_t left = live; left;) {
                const int r = __builtin_ctzll(left);
                const uint64_t behind = ~0ull << r << 1;
                if (!CTL || control(r, applied, nbase + uint64_t(k))) {
                    applied |= 1ull << r;
#pragma unroll
                    for (int h = 0; h < RPL; ++h) fm[h] = 0u;
                    pays(r);
                    const uint32_t on = uniform(PT[r * kProbeWords + 7]);
                    if (on) {
                        write(on, 1ull << r, fm, false, Py, ch);
#pragma unroll
                        for (int h = 0; h < RPL; ++h) Dc[h] |= ch[h];
                        if (r + 1 < Rt) match(ch, r + 1 - kMoveRules);
                    }
                }
                left = live & behind;
            }
#pragma unroll
            for (int h = 0; h < RPL; ++h) {
                D[h] = Dc[h];
                Fl[h] = ((lvoted >> C) & 1u) ? (rw[h] ? F[yr[h]] : 0u) : Fy[h];
            }
        } else {
            if (g == 0) {
#pragma unroll
                for (int h = 0; h < RPL; ++h)
                    if (rw[h]) F[yr[h]] = Fy[h];
            }
            next_rows<RPL>(Fy, Fn, y);
            // the four moves (rules 0..3: right, left, down, up) and their votes on the player
            // plane
            uint32_t m0[RPL], m1[RPL], m2[RPL], m3[RPL], m2p[RPL], m3p[RPL], pnew[RPL];
#pragma unroll
            for (int h = 0; h < RPL; ++h) {
                m0[h] = Py[h] & (Fy[h] >> 1) & ~(Wy[h] >> 1) & cm1;
                m1[h] = Fy[h] & ~Wy[h] & (Py[h] >> 1) & cm1;
                m2[h] = Py[h] & Fn[h] & ~Wn[h] & vrow2[h];
                m3[h] = Fy[h] & ~Wy[h] & Pn[h] & vrow2[h];
            }
            prev_rows<RPL>(m2, m2p, y);
            prev_rows<RPL>(m3, m3p, y);
            uint32_t both = 0u;
#pragma unroll
            for (int h = 0; h < RPL; ++h) {
                const uint32_t plus = (m0[h] << 1) | m1[h] | m2p[h] | m3[h];
                const uint32_t minus = m0[h] | (m1[h] << 1) | m2[h] | m3p[h];
                pnew[h] = (Py[h] | plus) & ~minus;
                both |= plus & minus;
            }
            // where some cell got votes of both signs (players moving into cells other players
            // leave), counted exactly: old + #plus > #minus
            if (__builtin_amdgcn_ballot_w64(both != 0u)) {
#pragma unroll
                for (int h = 0; h < RPL; ++h) {
                    uint32_t q[4] = {Py[h], 0u, 0u, 0u};
                    count4<4>(q, m0[h] << 1, m1[h], m2p[h], m3[h]);
                    count4<4>(q, ~m0[h], ~(m1[h] << 1), ~m2[h], ~m3p[h]);
                    pnew[h] = q[3] | (q[2] & (q[1] | q[0]));   // 5 or more of 9
                }
            }
            auto store_moves = [&]() AV_INLINE {  // the moves' match rows, for a recount
                if (g != 0) return;
#pragma unroll
                for (int h = 0; h < RPL; ++h) {
                    M[0 * MS + PAD + yr[h]] = m0[h];
                    M[1 * MS + PAD + yr[h]] = m1[h];
                    M[2 * MS + PAD + yr[h]] = m2[h];
                    M[3 * MS + PAD + yr[h]] = m3[h];
                }
            };
            if constexpr (HALVES) store_moves();   // (at once: held, they would spill registers)
            // every loaded rule's matches on this map
#pragma unroll
            for (int h = 0; h < RPL; ++h) {
                const uint32_t f = rw[h] ? Fy[h] : 0u;
                D[h] |= f ^ Fl[h];
                Fl[h] = f;
            }
            match(D, 0);
            uint64_t fired = live;
            if constexpr (CTL) {
                uint64_t applied = 0ull;
                for (uint64_t fr = fired; fr; fr &= fr - 1ull) {
                    const int r = __builtin_ctzll(fr);
                    if (control(r, applied, nbase + uint64_t(k))) applied |= 1ull << r;
                }
                fired = applied;
            }
            for (uint64_t fr = fired; fr; fr &= fr - 1ull) pays(__builtin_ctzll(fr));
            // the player plane by the moves' votes alone, from registers
            const bool player = (lvoted >> kChPlayer) & 1u;
            if (!player && g == 0) {
#pragma unroll
                for (int h = 0; h < RPL; ++h)
                    if (rw[h]) P2[yr[h]] = pnew[h];
            }
#pragma unroll
            for (int h = 0; h < RPL; ++h) D[h] = Py[h] ^ pnew[h];
            if (lvoted) {
                uint32_t ch[RPL];
                if (!HALVES && player) store_moves();
                lds_order();
                write(lvoted, fired, fm, true, pnew, ch);
#pragma unroll
                for (int h = 0; h < RPL; ++h) D[h] |= ch[h];
            }
#pragma unroll
            for (int h = 0; h < RPL; ++h) Py[h] = pnew[h];
        }

        // reward: the sum over a group's lanes
        if (__builtin_amdgcn_ballot_w64(rsum != 0)) rsum = int(group_sum(uint32_t(rsum)));
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
            live = 0ull;
#pragma unroll
            for (int h = 0; h < RPL; ++h) {
                D[h] = rw[h] ? ~0u : 0u;
                if (rw[h]) {
#pragma unroll 4
                    for (int c = g; c < C; c += kG) {
                        const size_t at = (size_t(c) * a.B + b) * H + yr[h];
                        P[c * PR + yr[h]] = a.row_bytes == 2
                                                ? uint32_t(static_cast<const uint16_t *>(a.init)[at])
                                                : static_cast<const uint32_t *>(a.init)[at];
                    }
                }
            }
            lds_order();
#pragma unroll
            for (int h = 0; h < RPL; ++h) {
                Py[h] = rw[h] ? P2[yr[h]] : 0u;
                Wy[h] = rw[h] ? P[kChWall * PR + yr[h]] : 0u;
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
        // the rows back as they were read, the lane's channel and row formed again from an
        // opaque copy of its index (kept from the set-up they would be spilled through the launch)
        int le = lane;
        asm volatile("" : "+v"(le));
        const int rcs = 64 / H, rcl = le / H, rrow = le - rcl * H;
        if (rcl < rcs) {
#pragma unroll 4
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

// LDS of a launch without the table's lists.
size_t group_base_bytes(int H, int W, int C, int rules_per_set, int max_pat_h, bool sequential,
                        bool control, bool random) {
    const int HR = group_rows(H), PR = group_plane_words(HR, pattern_rows(max_pat_h));
    return sizeof(uint32_t) *
           (size_t(C + 1) * PR + size_t(rules_per_set + 1) * PR * (control ? 2 : 1) +
            size_t(rules_per_set - kMoveRules + 1) * HR +
            size_t(group_head_words(rules_per_set, sequential ? C + 1 : C)) +
            (control ? size_t(3) * rules_per_set : 0) +
            (control && random ? size_t(H) * key_stride(W) + 32 : 0));
}

}  // namespace

bool group_eligible(int H, int W, int C, int rules_per_set, int max_pat_h, int max_pat_w) {
    if (H > 32 || W > 32) return false;
    // every vote a cell-channel gets comes from a distinct (rule, pattern cell): the 8-bit
    // counts of the exact write hold them (plus the old value) when there are at most 255
    if (long(rules_per_set) * max_pat_h * max_pat_w > 254) return false;
    // (rule masks are 64-bit; merged entries address rows of the stored and force planes in 12
    // bits: at most 1536 within these limits, and the LDS set at most 33 KiB)
    return rules_per_set <= 64 && C <= kMaxChan &&
           (C + 1) * group_plane_words(group_rows(H), pattern_rows(max_pat_h)) <=
               kMaxEntryOffset + 1 &&
           group_base_bytes(H, W, C, rules_per_set, max_pat_h, false, false, false) <=
               size_t(kLdsBudget);
}

bool group_mode_eligible(int H, int W, int C, int rules_per_set, int max_pat_h, int max_pat_w,
                         bool sequential, bool control, bool random) {
    if (H > 32 || W > 32 || (!sequential && !control)) return false;
    // as above; a vote list's places and a set's entries are 16-bit, and in sequential order only
    // one rule's votes are counted at a time
    const long cells = long(max_pat_h) * max_pat_w;
    const int PR = group_plane_words(group_rows(H), pattern_rows(max_pat_h));
    if (rules_per_set > 64 || (sequential ? 1 : rules_per_set) * cells > 254) return false;
    if (long(rules_per_set) * (C + 1) * cells > 0xFFFF || C + 1 > kMaxChan) return false;
    if (long(rules_per_set + 1) * PR * 4 > 0xFFFF) return false;
    return (C + 1) * PR <= kMaxEntryOffset + 1 &&
           group_base_bytes(H, W, C, rules_per_set, max_pat_h, sequential, control, random) <=
               size_t(kLdsBudget);
}

// Merges a rule's input entries (c | i << 8 | j << 16 | want << 24) per plane row and block of 8
// columns.
struct EntryMerger {
    int H, W, C, PR;
    std::vector<int32_t> place;                   // of (c, i, block) in out, -1
    std::vector<std::pair<float, uint32_t>> out;  // share of a typical map's cells passed, entry
    std::vector<uint64_t> keys;                   // the same in order: share's bits, entry

    EntryMerger(int H_, int W_, int C_, int PR_)
        : H(H_), W(W_), C(C_), PR(PR_), place(size_t(C_ + 1) * kMaxPat * 2, -1) {}

    // Those that accept the fewest cells of a typical map first: one tile per cell, a wall on three
    // cells in ten, the other tiles alike, one player (and its force) on the map.  (Only an order:
    // on maps of another kind the probe rejects less and results are the same.)
    void merge(const uint32_t *ent, int cnt) {
        const float few = 1.f / float(H * W), other = 0.7f / float(std::max(1, C - 2));
        out.clear();
        for (int e = 0; e < cnt; ++e) {
            const uint32_t c = ent[e] & 255u, i = (ent[e] >> 8) & 255u, j = (ent[e] >> 16) & 255u;
            int32_t &at = place[(c * kMaxPat + i) * 2 + (j >> 3)];
            if (at < 0) {                         // no column tested yet
                at = int32_t(out.size());
                out.push_back({1.f, (c * uint32_t(PR) + i) | ((j >> 3) << 12)});
            }
            const bool one = (ent[e] >> 24) & 1u;
            const float p = int(c) == C || int(c) == kChPlayer ? few : int(c) == kChWall ? 0.3f : other;
            auto &o = out[size_t(at)];
            o.second |= (1u << (j & 7u)) << (one ? 24 : 16);
            o.first *= one ? p : 1.f - p;
        }
        for (int e = 0; e < cnt; ++e)
            place[((ent[e] & 255u) * kMaxPat + ((ent[e] >> 8) & 255u)) * 2 + (((ent[e] >> 16) & 255u) >> 3)] = -1;
        // (equal ones by place, so that the order is one for every host; a share's bits order as it
        // does, being positive)
        keys.clear();
        for (const auto &o : out) {
            uint32_t share;
            std::memcpy(&share, &o.first, 4);
            keys.push_back((uint64_t(share) << 32) | o.second);
        }
        std::sort(keys.begin(), keys.end());
    }
};

void compile_group_tables(const GenericProgram &p, int H, int W, int C, int lists, int max_pat_h,
                          std::vector<uint32_t> &tab, int &stride, int &entry_words) {
    const int Rt = p.rules_per_set, C1 = C + 1;
    const int PAD = pattern_rows(max_pat_h) - 1, PR = group_plane_words(group_rows(H), PAD + 1);
    const int head = group_head_words(Rt, lists);
    EntryMerger em(H, W, C, PR);
    std::vector<uint32_t> merged;                 // every rule's entries, one after another
    std::vector<int32_t> counts;                  // and how many
    merged.reserve(p.match.size());
    size_t most_votes = 0, most_entries = 0;
    for (int s = 0; s < p.sets; ++s) {
        const size_t from = merged.size();
        for (int r = kMoveRules; r < Rt; ++r) {
            const RuleHdr &h = p.hdr[size_t(s) * Rt + r];
            em.merge(p.match.data() + size_t(s) * p.match_stride + h.match_off, h.match_cnt);
            for (const uint64_t key : em.keys) merged.push_back(uint32_t(key));
            counts.push_back(int32_t(em.keys.size()));
        }
        size_t votes = 0;
        for (int c = 0; c < lists; ++c) votes += size_t(p.votes[size_t(s) * C1 + c].cnt);
        most_votes = std::max(most_votes, votes);
        most_entries = std::max(most_entries, merged.size() - from);
    }
    entry_words = int((most_entries + 3) & ~size_t(3));
    stride = head + entry_words + int((most_votes + 4 + 3) & ~size_t(3));   // (four votes are read at a time)
    tab.assign(size_t(p.sets) * stride, 0u);
    const uint32_t *ent = merged.data();
    const int32_t *count = counts.data();
    for (int s = 0; s < p.sets; ++s) {
        uint32_t *pt = tab.data() + size_t(s) * stride, *rs = pt + (Rt + 1) * kProbeWords;
        uint32_t *gm = pt + head, *cv = gm + entry_words;
        int off = 0;
        for (int r = kMoveRules; r < Rt; ++r) {
            const RuleHdr &h = p.hdr[size_t(s) * Rt + r];
            const int cnt = *count++;
            std::copy(ent, ent + cnt, gm + off);
            uint32_t *row = pt + r * kProbeWords;
            // the first entries (a missing one always passes) and the anchors, columns 0 .. W - m
            // (~0 >> (32 - (W - m + 1))) of rows 0 .. H - n
            for (int e = 0; e < kProbeEntries; ++e) {
                row[e] = e < cnt ? ent[e] : kPassEntry;
                row[8 + e] = kProbeEntries + e < cnt ? ent[kProbeEntries + e] : kPassEntry;
            }
            const int cols = W - h.m + 1, rows = H - h.n + 1;
            row[4] = (cols >= 1 && rows >= 1) ? uint32_t(32 - cols) | (uint32_t(rows) << 8) : 0u;
            if (cnt > 2 * kProbeEntries) row[4] |= kMoreEntries;
            row[5] = uint32_t(off) | (uint32_t(cnt) << 16);
            row[6] = uint32_t(h.reward);
            row[7] = uint32_t(h.pad);
            off += cnt;
            ent += cnt;
        }
        // the channels' vote lists (each ordered by rule) and every rule's part of them
        uint32_t at = 0;
        for (int c = 0; c < lists; ++c) {
            const VoteList &vl = p.votes[size_t(s) * C1 + c];
            const uint32_t *v = p.vote.data() + size_t(s) * p.vote_stride + vl.off;
            for (int k = 0; k < vl.cnt; ++k, ++at) {
                const uint32_t r = v[k] & 255u, i = (v[k] >> 8) & 255u, j = (v[k] >> 16) & 255u;
                const bool minus = !((v[k] >> 24) & 1u);
                cv[at] = (r * uint32_t(PR) + uint32_t(PAD) - i) * 4u | (j << 16) | (minus ? kMinusVote : 0u);
                uint32_t &w = rs[c * Rt + int(r)];
                if (!((w >> 16) & 255u)) w = at;
                w += (1u << 16) + (minus ? 1u << 24 : 0u);
            }
        }
    }
}

namespace {
template <int RPL, int NJ>
void launch_mode(const StepArgs &a, size_t lds, int where, bool wide, hipStream_t s) {
    const dim3 grid(a.B), block(64);
    const bool ctl = a.ctl.active != 0, in = where == kLds;
#define AV_GROUP(SEQ, CTL, WHERE, WAVES) \
    hipLaunchKernelGGL((group_step<RPL, NJ, SEQ, CTL, WHERE, WAVES>), grid, block, lds, s, a)
    if (a.sequential && ctl) {
        if (in) AV_GROUP(true, true, kLds, 2);
        else AV_GROUP(true, true, kGlobal, 2);
    } else if (a.sequential) {
        if (in) AV_GROUP(true, false, kLds, 2);
        else AV_GROUP(true, false, kGlobal, 2);
    } else if (ctl) {
        if (in) AV_GROUP(false, true, kLds, 2);
        else AV_GROUP(false, true, kGlobal, 2);
    } else if (wide) {
        if (in) AV_GROUP(false, false, kLds, 2);
        else AV_GROUP(false, false, kGlobal, 2);
    } else {
        if (in) AV_GROUP(false, false, kLds, 4);
        else if (where == kEntries) AV_GROUP(false, false, kEntries, 4);
        else AV_GROUP(false, false, kGlobal, 4);
    }
#undef AV_GROUP
}

// SIMDs of the current device (4 per compute unit; device_wave_slots counts 8 waves on each).
int device_simds() {
    const long long slots = device_wave_slots();
    return slots > 0 ? int(slots / 8) : 1024;
}
}  // namespace

hipError_t launch_group_step(const StepArgs &step, hipStream_t s) {
    StepArgs a = step;
    a.max_pat_h = pattern_rows(a.max_pat_h);
    const int Rt = a.prog.rules_per_set, NC = a.sequential ? a.C + 1 : a.C;
    size_t lds = group_base_bytes(a.H, a.W, a.C, Rt, a.max_pat_h, a.sequential != 0,
                                  a.ctl.active != 0, a.ctl.random != 0);
    const size_t rest = sizeof(uint32_t) * size_t(a.prog.gtab_stride - group_head_words(Rt, NC));
    const size_t entries = sizeof(uint32_t) * size_t(a.prog.gentry_words);
    // Waves per SIMD the kernel's registers leave room for: two (256 registers) for batches that
    // need no more, and for sequential order and control, whose steps are long enough that
    // registers count for more; else four.
    const bool wide = a.B <= 2 * device_simds();
    const bool two = wide || a.sequential || a.ctl.active;
    // the lists go to LDS for launches of 16 steps or more, as far as they fit and leave room for
    // as many waves per CU (160 KiB of LDS) as the batch can use
    const size_t need = size_t(std::min(two ? 8 : 16, (a.B + 255) / 256));
    const size_t budget = std::min(size_t(kLdsBudget), kCuLds / need);
    int where = kGlobal;
    if (a.k >= kShortLaunch && lds + rest <= budget) {
        where = kLds;
        lds += rest;
    } else if (a.k >= kShortLaunch && !two && lds + entries <= budget) {
        where = kEntries;
        lds += entries;
    }
    const bool narrow = a.max_pat_w <= 3;
    if (group_rows(a.H) == 16) {
        if (narrow) launch_mode<1, 3>(a, lds, where, wide, s);
        else launch_mode<1, 8>(a, lds, where, wide, s);
    } else {
        if (narrow) launch_mode<2, 3>(a, lds, where, wide, s);
        else launch_mode<2, 8>(a, lds, where, wide, s);
    }
    return hipGetLastError();
}

}  // namespace av
