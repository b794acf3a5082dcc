// step.h -- one first-order transition on the radix-group sampling space
// (Sec. 4.1 hierarchical sampling: group by inverse transform over
// c_k 2^k, Eq. eq:group_prob; member uniformly, Eq. eq:pvp; rejection on
// the adjacency for dense groups, Sec. 5.1), and the chunked walk-id queue
// of the persistent kernels.  Shared by the walk kernels.
#pragma once
#include "dev.h"

namespace {

constexpr uint32_t PENDING = 0xFFFFFFFEu;
constexpr uint64_t NO_WALK = ~0ull;

// One round of SPEC dense-rejection attempts.  The attempt indices depend only
// on the random stream, not on the loaded words, so the SPEC loads are issued
// together and the dependent chain of a step shrinks from one load per attempt
// to one per round.  The accepted slot is the first accepting attempt in stream
// order, exactly as with one attempt at a time; words drawn for attempts after
// it are never used (every step, and every node2vec proposal, starts a fresh
// stream).  Returns PENDING when no
// attempt of the round accepts.
template <int SPEC>
__device__ __forceinline__ uint32_t dense_round(const uint64_t* __restrict__ edges, uint32_t d, uint32_t sel,
                                                RandStream& rs) {
    uint64_t e[SPEC];
#pragma unroll
    for (int a = 0; a < SPEC; ++a) e[a] = edges[rs_below32(rs, d)];
    uint32_t v = PENDING;
#pragma unroll
    for (int a = SPEC - 1; a >= 0; --a)
        if (((uint32_t)(e[a] >> 32) >> sel) & 1u) v = (uint32_t)e[a];
    return v;
}

// The decimal group of fixed-point biases (slot 0; Sec. 4.3): its members weigh
// their fractions q = weight mod 2^F.  A one-element group returns its member;
// otherwise a candidate is drawn uniformly from the group's list (listed types)
// or from the whole adjacency (dense) and accepted when the top F bits of the
// next random word are below its q.  Every member has q >= 1, so an attempt
// accepts with probability at least 2^-F (at least alpha % of that for the
// dense form); the attempt bound (2^24, with F <= 16) is never reached on a
// consistent structure and only keeps a corrupted one from spinning.
constexpr uint32_t DEC_MAX_ATTEMPTS = 1u << 24;

__device__ __forceinline__ uint32_t decimal_pick(const HdrCRef& h, const uint32_t* __restrict__ pool,
                                                 uint64_t adj, uint32_t d, uint32_t slot0, uint32_t onem,
                                                 GroupRule rule, RandStream& rs) {
    if (onem & 1u) return slot0;  // one member: its destination sits in the slot
    const uint64_t* __restrict__ edges = reinterpret_cast<const uint64_t*>(pool + adj);
    const uint32_t c0 = slot0;
    const uint32_t t = group_type(c0, d, rule);
    const uint32_t info = h[H_INFO];
    const uint32_t fm = (1u << rule.fbits) - 1u;
    const uint64_t lst = (uint64_t)info * LIST_UNIT_WORDS;
    for (uint32_t att = 0; att < DEC_MAX_ATTEMPTS; ++att) {
        const uint32_t i = type_listed(t) ? pool[lst + rs_below32(rs, c0)] : rs_below32(rs, d);
        const uint32_t x = rs_next32(rs) >> (32 - rule.fbits);
        const uint64_t e = edges[i];
        if (x < ((uint32_t)(e >> 32) & fm)) return (uint32_t)e;
    }
    return STOP_VERTEX;
}

// The group choice of a step at u (Sec. 4.1: group k with probability
// c_k 2^k / W, Eq. eq:group_prob).  Returns false at a vertex without out-edges.
// MODE 0 (integer biases, inverse transform): the ascending scan picks the k
// with prefix(k-1) <= r < prefix(k); with t = W - r that is the k with
// suffix(k+1) < t <= suffix(k), found from the top.  The header's first 64
// bytes hold the ten highest groups, so a step reads the rest of the slots
// only when t exceeds their total.  MODE 1 (fixed-point biases): integer
// groups F..31 ascending, the decimal group (slot 0) last, over all slots.
// MODE 2: the alias table picks the group; its slot comes from the first 64
// bytes when it is among the ten highest.
struct GroupPick {
    int sel;         // the group; -1: the decimal group (MODE 1), or an inconsistent header
    uint32_t csel;   // its count
    uint32_t raw;    // its slot word (a one-element group's destination)
    uint32_t d, onem, hi;
    uint32_t slot0;  // MODE 1: slot of group 0, the decimal group's count
    uint64_t adj;
};

template <int MODE>
__device__ __forceinline__ bool pick_group(const uint32_t* __restrict__ hdr, uint32_t u, RandStream& rs,
                                           GroupRule rule, GroupPick& g) {
    const HdrCRef h = hdr_ref(hdr, u);
    const uint4* h4 = reinterpret_cast<const uint4*>(h.hot);
    const uint4* x4 = reinterpret_cast<const uint4*>(h.cold + (H_SLOT10 - HDR_HOT));  // ranks 10..31, 2 spare words
    const uint4 q0 = h4[0], q1 = h4[1], q2 = h4[2], q3 = h4[3];
    g.d = q0.y;
    if (g.d == 0) return false;
    const uint64_t W = ((uint64_t)q0.w << 32) | q0.z;
    g.onem = q0.x;
    g.hi = q1.y >> H_HI_SHIFT;
    g.adj = ((uint64_t)(q1.y & H_ADJHI_MASK) << 32) | q1.x;
    g.sel = -1;
    g.csel = g.raw = g.slot0 = 0;
    uint32_t sl[32];  // sl[r]: slot of group hi - r
    sl[0] = q1.z; sl[1] = q1.w;
    sl[2] = q2.x; sl[3] = q2.y; sl[4] = q2.z; sl[5] = q2.w;
    sl[6] = q3.x; sl[7] = q3.y; sl[8] = q3.z; sl[9] = q3.w;
    if constexpr (MODE == 2) {
        // alias table: slot j from the top 5 bits of a word, then x < W against the slot's cut
        const uint32_t j = rs_next32(rs) >> 27;
        const uint4 e = rule.alias[(size_t)u * ALIAS_ENTRIES + j];
        const uint64_t x = rs_below64(rs, W);
        const uint32_t k = x < (((uint64_t)e.y << 32) | e.x) ? j : e.z;
        if (k > g.hi) return true;  // an empty group: only on an inconsistent structure
        const uint32_t r = g.hi - k;
        uint32_t raw = 0;
        if (r < 10) {
#pragma unroll
            for (int q = 0; q < 10; ++q)
                if ((uint32_t)q == r) raw = sl[q];
        } else {
            raw = h.slot(r);
        }
        g.sel = (int)k;
        g.raw = raw;
        g.csel = ((g.onem >> k) & 1u) ? 1u : raw;
    } else if constexpr (MODE == 1) {
        const uint4 q4 = x4[0], q5 = x4[1], q6 = x4[2], q7 = x4[3], q8 = x4[4], q9 = x4[5];
        sl[10] = q4.x; sl[11] = q4.y; sl[12] = q4.z; sl[13] = q4.w;
        sl[14] = q5.x; sl[15] = q5.y; sl[16] = q5.z; sl[17] = q5.w;
        sl[18] = q6.x; sl[19] = q6.y; sl[20] = q6.z; sl[21] = q6.w;
        sl[22] = q7.x; sl[23] = q7.y; sl[24] = q7.z; sl[25] = q7.w;
        sl[26] = q8.x; sl[27] = q8.y; sl[28] = q8.z; sl[29] = q8.w;
        sl[30] = q9.x; sl[31] = q9.y;
        // integer groups F..31 ascending (ranks descending), the decimal group last
        const uint64_t r = rs_below64(rs, W);
        uint64_t acc = 0;
#pragma unroll
        for (int q = 31; q >= 0; --q) {
            if ((uint32_t)q <= g.hi) {
                const uint32_t k = g.hi - (uint32_t)q;
                const uint32_t ck = ((g.onem >> k) & 1u) ? 1u : sl[q];
                if (k == 0) g.slot0 = sl[q];
                if (k >= rule.fbits) acc += shl32(ck, k);
                if (g.sel < 0 && r < acc) { g.sel = (int)k; g.csel = ck; g.raw = sl[q]; }
            }
        }
    } else {
        const uint64_t t = W - rs_below64(rs, W);  // in [1, W]
        uint64_t acc = 0;
#pragma unroll
        for (int q = 0; q < 10; ++q) {
            if (g.sel < 0 && (uint32_t)q <= g.hi) {
                const uint32_t k = g.hi - (uint32_t)q;
                const uint32_t ck = ((g.onem >> k) & 1u) ? 1u : sl[q];
                acc += shl32(ck, k);
                if (acc >= t) { g.sel = (int)k; g.csel = ck; g.raw = sl[q]; }
            }
        }
        if (g.sel < 0 && g.hi >= 10) {
            const uint4 q4 = x4[0], q5 = x4[1], q6 = x4[2], q7 = x4[3];
            sl[10] = q4.x; sl[11] = q4.y; sl[12] = q4.z; sl[13] = q4.w;
            sl[14] = q5.x; sl[15] = q5.y; sl[16] = q5.z; sl[17] = q5.w;
            sl[18] = q6.x; sl[19] = q6.y; sl[20] = q6.z; sl[21] = q6.w;
            sl[22] = q7.x; sl[23] = q7.y; sl[24] = q7.z; sl[25] = q7.w;
#pragma unroll
            for (int q = 10; q < 26; ++q) {
                if (g.sel < 0 && (uint32_t)q <= g.hi) {
                    const uint32_t k = g.hi - (uint32_t)q;
                    const uint32_t ck = ((g.onem >> k) & 1u) ? 1u : sl[q];
                    acc += shl32(ck, k);
                    if (acc >= t) { g.sel = (int)k; g.csel = ck; g.raw = sl[q]; }
                }
            }
            if (g.sel < 0 && g.hi >= 26) {
                const uint4 q8 = x4[4], q9 = x4[5];
                sl[26] = q8.x; sl[27] = q8.y; sl[28] = q8.z; sl[29] = q8.w;
                sl[30] = q9.x; sl[31] = q9.y;
#pragma unroll
                for (int q = 26; q < 32; ++q) {
                    if (g.sel < 0 && (uint32_t)q <= g.hi) {
                        const uint32_t k = g.hi - (uint32_t)q;
                        const uint32_t ck = ((g.onem >> k) & 1u) ? 1u : sl[q];
                        acc += shl32(ck, k);
                        if (acc >= t) { g.sel = (int)k; g.csel = ck; g.raw = sl[q]; }
                    }
                }
            }
        }
    }
    return true;
}

// One transition from u (no termination test).  Returns the next vertex or
// STOP_VERTEX for a vertex without out-edges.  MODE 0: integer biases, inverse
// transform over the groups; 1: fixed-point biases (rule.fbits > 0, decimal
// group taken last); 2: integer biases, alias table (rule.alias).  Each
// instance carries only its own selection code.
template <int SPEC, int MODE>
__device__ __forceinline__ uint32_t walk_step_body(const uint32_t* __restrict__ hdr, const uint32_t* __restrict__ pool,
                                                   uint32_t u, RandStream& rs, GroupRule rule) {
    GroupPick g;
    if (!pick_group<MODE>(hdr, u, rs, rule, g)) return STOP_VERTEX;
    if (MODE == 1 && g.sel < 0)
        return decimal_pick(hdr_ref(hdr, u), pool, g.adj, g.d, g.slot0, g.onem, rule, rs);
    if (g.sel < 0) return STOP_VERTEX;  // only on an inconsistent header
    if ((g.onem >> g.sel) & 1u) return g.raw;  // one-element group: the step ends in the header
    const uint64_t* __restrict__ edges = reinterpret_cast<const uint64_t*>(pool + g.adj);
    const uint32_t t = group_type(g.csel, g.d, rule);
    if (t == GT_DENSE) {
        // rejection on the whole neighbor list: accept a slot whose weight has
        // bit sel.  Acceptance is above alpha % per attempt, so the bound is
        // never reached on a consistent structure; it only keeps a corrupted
        // one from spinning forever.
        for (uint32_t att = 0; att < (1u << 16); att += SPEC) {
            const uint32_t v = dense_round<SPEC>(edges, g.d, (uint32_t)g.sel, rs);
            if (v != PENDING) return v;
        }
        return STOP_VERTEX;
    }
    const uint32_t info = hdr_ref(hdr, u)[H_INFO + (uint32_t)g.sel];
    const uint32_t i = pool[(uint64_t)info * LIST_UNIT_WORDS + rs_below32(rs, g.csel)];
    return pool[g.adj + 2ull * i];
}

// The same transition word by word from block blk0 of the stream (skip words passed
// over), as one loop around one Philox block: small code and few registers, for
// the rare steps that the lean kernels below hand over.
template <int MODE>
__device__ __forceinline__ uint32_t odd_step(const uint32_t* __restrict__ hdr, const uint32_t* __restrict__ pool,
                                             uint32_t u, uint64_t seed, uint64_t id, uint32_t s, uint32_t blk0,
                                             uint32_t skip, GroupRule rule) {
    const HdrCRef h = hdr_ref(hdr, u);
    const uint32_t d = h[H_DEG], onem = h[H_ONEMASK], hi = hdr_hi(h);
    if (d == 0) return STOP_VERTEX;
    const uint64_t W = ((uint64_t)h[H_WHI] << 32) | h[H_WLO], adj = hdr_adj(h);
    const uint64_t* __restrict__ edges = reinterpret_cast<const uint64_t*>(pool + adj);
    // what the next word is: the alias slot, the group draw's halves, then a member draw of one of
    // the forms below; an index draw of the decimal group is followed by its acceptance word
    enum { ALIAS, HIGH, LOW, DENSE, LIST, DEC_INDEX, DEC_TEST };
    uint32_t want = MODE == 2 ? ALIAS : HIGH, b0 = 0, b1 = 0, b2 = 0, b3 = 0, slot = 0, sel = 0, n = 0, att = 0;
    uint64_t x = 0, list = 0, e = 0;
#pragma unroll 1
    for (uint32_t pos = skip;; ++pos) {
        if (pos == skip || (pos & 3u) == 0)
            philox_uniform((uint32_t)id, (uint32_t)(id >> 32), s, blk0 + (pos >> 2), seed, b0, b1, b2, b3);
        const uint32_t w = (pos & 2u) ? ((pos & 1u) ? b3 : b2) : ((pos & 1u) ? b1 : b0);
        if (want == ALIAS) {
            slot = w >> 27;
            want = HIGH;
        } else if (want == HIGH) {
            x = (uint64_t)w << 32;
            want = LOW;
        } else if (want == LOW) {
            x |= w;
            want = HIGH;
            const uint64_t low = x * W;
            if (low < W && low < (0ull - W) % W) continue;  // Lemire: draw again
            const uint64_t r = __umul64hi(x, W);
            sel = 32u;
            if constexpr (MODE == 2) {
                const uint4 a = rule.alias[(size_t)u * ALIAS_ENTRIES + slot];
                const uint32_t k = r < (((uint64_t)a.y << 32) | a.x) ? slot : a.z;
                if (k <= hi) sel = k;
            } else {
                uint64_t acc = 0;
#pragma unroll 1
                for (uint32_t k = MODE == 1 ? rule.fbits : 0u; k <= hi && sel == 32u; ++k) {
                    acc += shl32(slot_count(h.slot(hi - k), onem, k), k);
                    if (r < acc) sel = k;
                }
            }
            const bool dec = MODE == 1 && sel == 32u;
            if (dec) sel = 0;
            if (sel == 32u) return STOP_VERTEX;  // only on an inconsistent header
            const uint32_t raw = h.slot(hi - sel);
            if ((onem >> sel) & 1u) return raw;
            const uint32_t t = group_type(raw, d, rule);
            list = (uint64_t)h[H_INFO + sel] * LIST_UNIT_WORDS;
            n = type_listed(t) ? raw : d;
            want = dec ? DEC_INDEX : (type_listed(t) ? LIST : DENSE);
            if (dec && !type_listed(t)) list = ~0ull;
        } else if (want == DEC_TEST) {
            // accepted when the top F bits are below the fraction (see decimal_pick)
            const uint32_t fm = (1u << rule.fbits) - 1u;
            if ((w >> (32 - rule.fbits)) < ((uint32_t)(e >> 32) & fm)) return (uint32_t)e;
            if (++att >= DEC_MAX_ATTEMPTS) return STOP_VERTEX;
            want = DEC_INDEX;
        } else {
            const uint64_t m = (uint64_t)w * n;
            const uint32_t low = (uint32_t)m;
            if (low < n && low < (0u - n) % n) continue;
            const uint32_t i = (uint32_t)(m >> 32);
            if (want == DENSE) {
                const uint64_t y = edges[i];
                if (((uint32_t)(y >> 32) >> sel) & 1u) return (uint32_t)y;
                if (++att >= (1u << 16)) return STOP_VERTEX;
            } else {
                e = edges[list == ~0ull ? i : pool[list + i]];
                if (want == LIST) return (uint32_t)e;
                want = DEC_TEST;
            }
        }
    }
}

// ---------------------------------------------------------------------------
// The lean step.  walk_step_body above draws word by word from a RandStream,
// whose refills sit behind tests that the lanes of a wave answer differently:
// a wave then runs Philox several times per step, each for a few lanes.  Here a
// lane computes one whole block per iteration, all lanes together, and the
// words have fixed places in it: the termination word (TERM, walks that have
// one), the alias slot (MODE 2), the 64-bit group draw, then one word per dense
// attempt.  What a draw needs beyond that is rare and goes through
// odd_step: a group draw in Lemire's biased zone (probability
// W / 2^64) and a redraw of a list position.  The sums of vertices of 2^21 edges
// and more pass 32 bits: a lane's own step takes them in 64 (wide_rank; as odd
// steps, a hub of 3 x 2^20 edges took 3000 x 1000 PageRank walks 2040 us, now
// 1090), the lanes that share a walk go through odd_step there.
// ---------------------------------------------------------------------------
constexpr uint32_t LEAN_MAX_DEG = 1u << 21;

// The group choice of the hot line by 32-bit sums.  With t = W - r (r the draw),
// the group is the first rank q whose total from the top, A_q 2^(hi - q) with
// A_q = 2 A_(q-1) + c_q, reaches t; that is A_q > (t - 1) >> (hi - q).  A_q stays
// below d 2^10 < 2^31 for ten ranks.  A draw below the ten highest groups
// continues with the remainder, ten ranks at a time.  Returns the rank (32: none,
// only on an inconsistent header); raw: its slot.
__device__ __forceinline__ uint32_t lean_rank(const HdrCRef& h, const uint32_t (&sl)[HOT_RANKS], uint64_t tm1,
                                              uint32_t hi, uint32_t onem, uint32_t& raw) {
    uint32_t om = onem << (31 - hi);  // bit 31 - q: rank q is a one-element group
    const uint32_t t9 = hi >= 9 ? shr64_lo(tm1, hi - 9) : (uint32_t)tm1 << (9 - hi);
    uint32_t A = 0, cnt = 0;
    raw = sl[0];
#pragma unroll
    for (int q = 0; q < HOT_RANKS; ++q) {
        A = 2 * A + ((om >> (31 - q)) & 1u ? 1u : sl[q]);
        const bool below = A <= (t9 >> (9 - q));
        cnt += below ? 1u : 0u;
        if (q + 1 < HOT_RANKS) raw = below ? sl[q + 1 < HOT_RANKS ? q + 1 : 0] : raw;
    }
    if (cnt < HOT_RANKS) return cnt;
    uint64_t rest = tm1;
    uint32_t top = hi;  // group of the chunk's first rank
    for (uint32_t base = HOT_RANKS; base <= hi; base += HOT_RANKS) {
        rest -= shl32(A, top - 9);  // the ranks so far; top >= 10 here
        top = hi - base;
        om <<= HOT_RANKS;
        uint32_t x[HOT_RANKS];
        const uint2* c2 = reinterpret_cast<const uint2*>(h.cold + (H_SLOT10 - HDR_HOT - HOT_RANKS) + base);
#pragma unroll
        for (int q = 0; q < HOT_RANKS / 2; ++q) {
            const uint2 y = c2[q];
            x[2 * q] = y.x;
            x[2 * q + 1] = y.y;
        }
        const uint32_t t = top >= 9 ? shr64_lo(rest, top - 9) : (uint32_t)rest << (9 - top);
        uint32_t n = 0;
        A = 0;
        raw = x[0];
#pragma unroll
        for (int q = 0; q < HOT_RANKS; ++q) {
            const uint32_t c = base + q > hi ? 0u : ((om >> (31 - q)) & 1u ? 1u : x[q]);
            A = 2 * A + c;
            const bool below = A <= (t >> (9 - q));
            n += below ? 1u : 0u;
            if (q + 1 < HOT_RANKS) raw = below ? x[q + 1 < HOT_RANKS ? q + 1 : 0] : raw;
        }
        if (n < HOT_RANKS) return base + n;
    }
    return 32u;
}

// The same choice in 64 bits, for vertices of LEAN_MAX_DEG edges and more: rank by rank from the top.
__device__ __forceinline__ uint32_t wide_rank(const HdrCRef& h, const uint32_t (&sl)[HOT_RANKS], uint64_t tm1,
                                              uint32_t hi, uint32_t onem, uint32_t& raw) {
    const uint32_t om = onem << (31 - hi);
    uint64_t rest = tm1;
    uint32_t rank = 32u;
    raw = 0;
#pragma unroll
    for (int q = 0; q < HOT_RANKS; ++q) {
        if (rank == 32u && (uint32_t)q <= hi) {
            const uint64_t T = shl32((om >> (31 - q)) & 1u ? 1u : sl[q], hi - q);
            if (rest < T) {
                rank = q;
                raw = sl[q];
            } else {
                rest -= T;
            }
        }
    }
#pragma unroll 1
    for (uint32_t q = HOT_RANKS; rank == 32u && q <= hi; ++q) {
        const uint32_t c = h.slot(q);
        const uint64_t T = shl32((om >> (31 - q)) & 1u ? 1u : c, hi - q);
        if (rest < T) {
            rank = q;
            raw = c;
        } else {
            rest -= T;
        }
    }
    return rank;
}

// type of a group known to have members and not to be one-element (d < LEAN_MAX_DEG, and any d)
__device__ __forceinline__ bool lean_dense(uint32_t c, uint32_t d, GroupRule r) {
    return r.adaptive && c * 100u > r.alpha * d;
}
__device__ __forceinline__ bool wide_dense(uint32_t c, uint32_t d, GroupRule r) {
    return r.adaptive && (uint64_t)c * 100u > (uint64_t)r.alpha * d;
}

// What a step comes to after its group choice.
enum : uint32_t { LK_DONE = 0, LK_DENSE = 1, LK_LIST = 2, LK_ODD = 3, LK_DEC = 4 };
struct LeanPick {
    uint32_t kind;  // LK_DONE: the next vertex is v; LK_ODD: take the step through odd_step; LK_DEC: a member of
                    // the decimal group (MODE 1), by decimal_draw
    uint32_t v, sel, csel, d;
    uint64_t adj;
};

// The header words a group choice needs, loaded ahead of their use.
struct HotLine {
    uint4 q0, q1, q2, q3;
};
__device__ __forceinline__ HotLine load_hot(const uint32_t* __restrict__ hdr, uint32_t u) {
    const uint4* h4 = reinterpret_cast<const uint4*>(hdr_ref(hdr, u).hot);
    return HotLine{h4[0], h4[1], h4[2], h4[3]};
}

// The alias entry that word a of the stream names (MODE 2), loaded beside the header.
template <int MODE>
__device__ __forceinline__ uint4 load_alias(bool want, uint32_t u, uint32_t a, GroupRule rule) {
    uint4 e = make_uint4(0u, 0u, 0u, 0u);
    if constexpr (MODE == 2)
        if (want) e = rule.alias[(size_t)u * ALIAS_ENTRIES + (a >> 27)];
    return e;
}

// Group choice from the words of the step's stream behind the termination word:
// MODE 0 and 1: x = a << 32 | b; MODE 2: slot from a with its entry e, x = b << 32 | c.
// WIDE, for large vertices: WIDE_ODD none, they go through odd_step; WIDE_FORK a branch with sums of their own;
// WIDE_TAIL those sums behind the common ones, over what these have come to.
enum { WIDE_ODD = 0, WIDE_FORK = 1, WIDE_TAIL = 2 };
template <int MODE, int WIDE>
__device__ __forceinline__ LeanPick lean_pick(const uint32_t* __restrict__ hdr, uint32_t u, const HotLine& q,
                                              uint32_t a, uint32_t b, uint32_t c, const uint4& e, GroupRule rule) {
    LeanPick p;
    p.kind = LK_DONE;
    p.v = STOP_VERTEX;
    p.sel = p.csel = 0;
    p.d = q.q0.y;
    p.adj = ((uint64_t)(q.q1.y & H_ADJHI_MASK) << 32) | q.q1.x;
    if (p.d == 0) return p;
    const HdrCRef h = hdr_ref(hdr, u);
    const uint64_t W = ((uint64_t)q.q0.w << 32) | q.q0.z;
    const uint32_t onem = q.q0.x, hi = q.q1.y >> H_HI_SHIFT;
    const uint64_t x = MODE == 2 ? ((uint64_t)b << 32) | c : ((uint64_t)a << 32) | b;
    if (x * W < W || (MODE != 2 && WIDE == WIDE_ODD && p.d >= LEAN_MAX_DEG)) {
        p.kind = LK_ODD;
        return p;
    }
    const uint64_t r = __umul64hi(x, W);
    const uint32_t sl[HOT_RANKS] = {q.q1.z, q.q1.w, q.q2.x, q.q2.y, q.q2.z, q.q2.w, q.q3.x, q.q3.y, q.q3.z, q.q3.w};
    uint32_t rank, raw;
    uint64_t tm1 = 0;
    if constexpr (MODE == 0) {
        tm1 = W - 1 - r;
        if (WIDE != WIDE_FORK || p.d < LEAN_MAX_DEG) rank = lean_rank(h, sl, tm1, hi, onem, raw);
        else rank = wide_rank(h, sl, tm1, hi, onem, raw);
    } else if constexpr (MODE == 2) {
        const uint32_t k = r < (((uint64_t)e.y << 32) | e.x) ? a >> 27 : e.z;
        rank = k > hi ? 32u : hi - k;  // above hi: only on an inconsistent structure
        raw = 0;
        if (rank < HOT_RANKS) {
#pragma unroll
            for (int i = 0; i < HOT_RANKS; ++i)
                if ((uint32_t)i == rank) raw = sl[i];
        } else if (rank < 32u) {
            raw = h.slot(rank);
        }
    } else {
        // integer groups F..31 ascending, the decimal group last: from the top, with I the integer
        // groups' total, a draw r >= I picks the decimal group and t = I - r picks as in MODE 0
        const uint32_t nint = hi + 1 > rule.fbits ? hi + 1 - rule.fbits : 0u;  // ranks of integer groups
        const uint32_t om = onem << (31 - hi);  // bit 31 - i: rank i is a one-element group
        uint2 y[11];                            // the cold ranks
        if (nint > HOT_RANKS) {
            const uint2* c2 = reinterpret_cast<const uint2*>(h.cold + (H_SLOT10 - HDR_HOT));
#pragma unroll
            for (int i = 0; i < 11; ++i) y[i] = c2[i];
        }
        uint64_t I = 0;
        if (WIDE == WIDE_ODD || p.d < LEAN_MAX_DEG) {
            // summed in 32 bits as in lean_rank, eleven ranks at a time past the hot line (d 2^11 is below 2^32)
            uint32_t A = 0;
#pragma unroll
            for (int i = 0; i < HOT_RANKS; ++i)
                if ((uint32_t)i < nint) A = 2 * A + ((om >> (31 - i)) & 1u ? 1u : sl[i]);
            I = shl32(A, hi + 1 - min(nint, (uint32_t)HOT_RANKS));
            if (nint > HOT_RANKS) {
#pragma unroll
                for (int b0 = 0; b0 < 22; b0 += 11) {
                    A = 0;
#pragma unroll
                    for (int i = b0; i < b0 + 11; ++i) {
                        const uint32_t c = i & 1 ? y[i / 2].y : y[i / 2].x;
                        if ((uint32_t)(i + HOT_RANKS) < nint)
                            A = 2 * A + ((om >> (31 - HOT_RANKS - i)) & 1u ? 1u : c);
                    }
                    if (nint > (uint32_t)(b0 + HOT_RANKS))
                        I += shl32(A, hi + 1 - min(nint, (uint32_t)(b0 + 11 + HOT_RANKS)));
                }
            }
        } else {
#pragma unroll
            for (int i = 0; i < 32; ++i) {
                const uint32_t c = i < HOT_RANKS ? sl[i < HOT_RANKS ? i : 0]
                                                 : ((i & 1) ? y[i < HOT_RANKS ? 0 : (i - HOT_RANKS) / 2].y
                                                            : y[i < HOT_RANKS ? 0 : (i - HOT_RANKS) / 2].x);
                if ((uint32_t)i < nint) I = 2 * I + ((om >> (31 - i)) & 1u ? 1u : c);
            }
            I <<= rule.fbits;  // the last integer rank is group F (none: I is 0)
        }
        if (r >= I) {
            // the decimal group, slot 0; a member alone is the step's end
            raw = sl[0];
#pragma unroll
            for (int i = 1; i < HOT_RANKS; ++i)
                if ((uint32_t)i == hi) raw = sl[i];
            if (hi >= HOT_RANKS) raw = h.slot(hi);
            p.csel = raw;
            p.v = raw;
            p.kind = (onem & 1u) ? LK_DONE : LK_DEC;
            return p;
        }
        // ranks below the integer groups are not reached: their groups' totals lie beyond t
        tm1 = I - 1 - r;
        if (WIDE != WIDE_FORK || p.d < LEAN_MAX_DEG) rank = lean_rank(h, sl, tm1, hi, onem, raw);
        else rank = wide_rank(h, sl, tm1, hi, onem, raw);
    }
    bool dense = lean_dense(raw, p.d, rule);
    if ((WIDE == WIDE_TAIL || MODE == 2) && p.d >= LEAN_MAX_DEG) {
        if (MODE != 2) rank = wide_rank(h, sl, tm1, hi, onem, raw);
        dense = wide_dense(raw, p.d, rule);
    }
    if (rank > hi) return p;  // only on an inconsistent header
    p.sel = hi - rank;
    if ((onem >> p.sel) & 1u) {
        p.v = raw;  // one-element group: the step ends in the header
        return p;
    }
    p.csel = raw;
    if (WIDE == WIDE_FORK && MODE != 2 && p.d >= LEAN_MAX_DEG) dense = wide_dense(raw, p.d, rule);
    p.kind = dense ? LK_DENSE : LK_LIST;
    return p;
}

// Word w as a draw on [0, n) (Lemire): true when it is rejected, else i is the draw.
__device__ __forceinline__ bool lean_reject(uint32_t w, uint32_t n, uint32_t& i) {
    const uint64_t m = (uint64_t)w * n;
    i = (uint32_t)(m >> 32);
    const uint32_t low = (uint32_t)m;
    return low < n && low < (0u - n) % n;
}

// A member of the decimal group (decimal_pick), the words taken from position HEAD of the step's stream on, whose
// first block is z, one after the other: for the lanes that share a walk.
template <uint32_t HEAD>
__device__ __forceinline__ uint32_t decimal_draw(const uint32_t* __restrict__ hdr, const uint32_t* __restrict__ pool,
                                                 uint32_t u, const LeanPick& p, uint64_t seed, uint64_t id, uint32_t s,
                                                 uint32_t blk0, uint32_t z0, uint32_t z1, uint32_t z2, uint32_t z3,
                                                 GroupRule rule) {
    const bool dense = wide_dense(p.csel, p.d, rule);
    const uint32_t n = dense ? p.d : p.csel;
    const uint32_t* __restrict__ L =
        pool + (dense ? 0ull : (uint64_t)hdr_ref(hdr, u)[H_INFO] * LIST_UNIT_WORDS);
    const uint64_t* __restrict__ edges = reinterpret_cast<const uint64_t*>(pool + p.adj);
    const uint32_t fm = (1u << rule.fbits) - 1u;
    uint32_t pos = HEAD;
    auto next = [&]() {
        if ((pos & 3u) == 0)
            philox_uniform((uint32_t)id, (uint32_t)(id >> 32), s, blk0 + (pos >> 2), seed, z0, z1, z2, z3);
        const uint32_t w = (pos & 2u) ? ((pos & 1u) ? z3 : z2) : ((pos & 1u) ? z1 : z0);
        ++pos;
        return w;
    };
#pragma unroll 1
    for (uint32_t att = 0; att < DEC_MAX_ATTEMPTS;) {
        uint32_t i;
        if (lean_reject(next(), n, i)) continue;
        if (!dense) i = L[i];
        const uint64_t e = edges[i];
        const uint32_t x = next() >> (32 - rule.fbits);
        if (x < ((uint32_t)(e >> 32) & fm)) return (uint32_t)e;
        ++att;
    }
    return STOP_VERTEX;
}

// A walk's step in progress in one lane.  Between iterations only dense steps and
// draws from the decimal group whose attempts have all been rejected so far remain.
struct LaneStep {
    uint64_t adj;
    uint32_t d, sel;
    uint32_t blk;    // next block of the step's stream
    bool pending;
    // the decimal group (MODE 1): sel is DEC_SEL, d the bound of its draws
    uint32_t info;   // its list's block, NO_LIST: the whole adjacency
    uint64_t carry;  // TERM = 1: the candidate whose acceptance word is the next block's first
};
constexpr uint32_t DEC_SEL = 32u, NO_LIST = 0xFFFFFFFFu;

// Up to four attempts of a dense step from one block's words (the first `skip` of
// them are none), SPEC loads at a time; PENDING when none is accepted.
template <int SPEC>
__device__ __forceinline__ uint32_t lane_attempts(const uint32_t* __restrict__ pool, const LaneStep& ls, uint32_t w0,
                                                  uint32_t w1, uint32_t w2, uint32_t w3, uint32_t skip) {
    const uint64_t* __restrict__ edges = reinterpret_cast<const uint64_t*>(pool + ls.adj);
    const uint32_t w[4] = {w0, w1, w2, w3};
    uint32_t v = PENDING;
#pragma unroll
    for (int r = 0; r < 4; r += SPEC) {
        if (v == PENDING && skip < (uint32_t)(r + SPEC)) {
            uint64_t e[SPEC];
            bool ok[SPEC];
#pragma unroll
            for (int a = 0; a < SPEC; ++a) {
                uint32_t i;
                ok[a] = !lean_reject(w[r + a], ls.d, i) && skip <= (uint32_t)(r + a);
                e[a] = 0;
                if (ok[a]) e[a] = edges[i];
            }
#pragma unroll
            for (int a = SPEC - 1; a >= 0; --a)
                if (ok[a] && (((uint32_t)(e[a] >> 32) >> ls.sel) & 1u)) v = (uint32_t)e[a];
        }
    }
    return v;
}

// A block's words for a draw from the decimal group (decimal_pick): pairs of an index and an acceptance word.  A
// step's pairs begin at its third word, or, behind a termination word, at its fourth, so that they straddle the
// blocks there and a candidate is carried over.  The first `skip` words of the block are none of them.  An index to
// be drawn again would shift the pairs: odd.
template <int TERM>
__device__ __forceinline__ uint32_t lane_decimal(const uint32_t* __restrict__ pool, LaneStep& ls, uint32_t fbits,
                                                 uint32_t w0, uint32_t w1, uint32_t w2, uint32_t w3, uint32_t skip,
                                                 bool& odd) {
    const uint64_t* __restrict__ edges = reinterpret_cast<const uint64_t*>(pool + ls.adj);
    auto fetch = [&](uint32_t w) {
        uint32_t i;
        if (lean_reject(w, ls.d, i)) {
            odd = true;
            return (uint64_t)0;
        }
        if (ls.info != NO_LIST) i = pool[(uint64_t)ls.info * LIST_UNIT_WORDS + i];
        return edges[i];
    };
    const uint32_t fm = (1u << fbits) - 1u;
    auto pass = [&](uint32_t w, uint64_t e) { return (w >> (32 - fbits)) < ((uint32_t)(e >> 32) & fm); };
    uint64_t e;
    if constexpr (TERM) {
        if (skip == 0) {
            if (pass(w0, ls.carry)) return (uint32_t)ls.carry;
            e = fetch(w1);
            if (pass(w2, e)) return (uint32_t)e;
        }
        if (!odd) ls.carry = fetch(w3);
    } else {
        if (skip == 0) {
            e = fetch(w0);
            if (pass(w1, e)) return (uint32_t)e;
        }
        if (!odd) {
            e = fetch(w2);
            if (pass(w3, e)) return (uint32_t)e;
        }
    }
    return PENDING;
}

// One iteration of a lane's step at u: a new step (ls.pending false) or more
// attempts of the one in progress, from one Philox block either way.  Returns
// PENDING when the step goes on, STOP_VERTEX at a vertex without out-edges,
// else the next vertex; `ended` when the termination word (TERM = 1) ends the
// walk before the step.  blk0: first block of the step's stream (node2vec
// proposals).  With WAVE a dense step of a vertex of degree >= wave_deg is
// returned as PENDING with serve set, ls.blk * 4 - left words of its stream used.
// SPEC attempts are loaded together.  WIDE as in lean_pick: the fork costs the walks that never meet a large vertex
// 2 % in the kernels with a termination word and in node2vec, the tail 14 % in the DeepWalk kernel (at 72 registers
// it spills 16).  All lanes of the wave call.
template <int SPEC, int MODE, int TERM, bool WAVE, int WIDE>
__device__ __forceinline__ uint32_t lane_advance(const uint32_t* __restrict__ hdr, const uint32_t* __restrict__ pool,
                                                 bool act, uint32_t u, LaneStep& ls, uint64_t seed, uint64_t id,
                                                 uint32_t s, uint32_t blk0, uint32_t thr, GroupRule rule,
                                                 uint32_t wave_deg, bool& ended, bool& serve, uint32_t& left) {
    constexpr uint32_t HEAD = TERM + (MODE == 2 ? 3 : 2);  // words before the first attempt
    ended = serve = false;
    left = 0;
    uint32_t v = PENDING;
    const bool begin = act && !ls.pending;
    HotLine q;
    if (begin) q = load_hot(hdr, u);
    uint32_t w0 = 0, w1 = 0, w2 = 0, w3 = 0;
    if (act) {
        const uint32_t blk = begin ? 0u : ls.blk;
        philox_uniform((uint32_t)id, (uint32_t)(id >> 32), s, blk0 + blk, seed, w0, w1, w2, w3);
        ls.blk = blk + 1;
    }
    const uint4 al = load_alias<MODE>(begin && !(TERM && w0 < thr), u, TERM ? w1 : w0, rule);
    uint32_t skip = act ? 0u : 4u;  // words of the block that are no attempts
    uint32_t lcnt = 0, linfo = 0;
    bool odd = false;
    if (begin) {
        skip = HEAD;
        if (TERM && w0 < thr) {
            ended = true;
            skip = 4;
        } else {
            const LeanPick p = TERM ? lean_pick<MODE, WIDE>(hdr, u, q, w1, w2, w3, al, rule)
                                    : lean_pick<MODE, WIDE>(hdr, u, q, w0, w1, w2, al, rule);
            if (p.kind == LK_DENSE) {
                ls.adj = p.adj; ls.d = p.d; ls.sel = p.sel; ls.pending = true;
                if (WAVE && p.d >= wave_deg) {
                    serve = true;
                    left = 4 - HEAD;
                }
            } else if (p.kind == LK_LIST) {
                ls.adj = p.adj;
                lcnt = p.csel;
                linfo = hdr_ref(hdr, u)[H_INFO + p.sel];  // used behind the attempts of the other lanes
            } else if (p.kind == LK_ODD) {
                odd = true;
            } else if (MODE == 1 && p.kind == LK_DEC) {
                const bool dense = wide_dense(p.csel, p.d, rule);
                ls.adj = p.adj; ls.d = dense ? p.d : p.csel; ls.sel = DEC_SEL; ls.pending = true;
                ls.info = dense ? NO_LIST : hdr_ref(hdr, u)[H_INFO];
            } else {
                v = p.v;
            }
        }
    }
    if (HEAD > 3 && begin && ((ls.pending && !serve) || lcnt)) {
        // the first block is used up: the member's words come from the next one
        philox_uniform((uint32_t)id, (uint32_t)(id >> 32), s, blk0 + ls.blk, seed, w0, w1, w2, w3);
        ++ls.blk;
        skip = 0;
    }
    if (ls.pending && act && !serve) {
        auto attempts = [&](uint32_t none) {
            if (MODE == 1 && ls.sel == DEC_SEL)
                return lane_decimal<TERM>(pool, ls, rule.fbits, w0, w1, w2, w3, none, odd);
            return lane_attempts<SPEC>(pool, ls, w0, w1, w2, w3, none);
        };
        v = attempts(skip);
        if (HEAD == 3 && v == PENDING && (MODE != 1 || !odd)) {
            // block 0 has one word left for the first attempt; a second block here spares every other step an
            // iteration of its own
            philox_uniform((uint32_t)id, (uint32_t)(id >> 32), s, blk0 + ls.blk, seed, w0, w1, w2, w3);
            ++ls.blk;
            v = attempts(0u);
        }
        // 2^14 blocks without an acceptance hold a few attempts less than the 2^16 that end a step (a group of a
        // few members in a large vertex is dense where alpha is next to nothing): odd_step counts them
        odd |= v == PENDING && ls.blk >= (1u << 14);
        if (v != PENDING || odd) ls.pending = false;
    }
    if (lcnt) {
        // the list position's word follows the group draw
        const uint32_t w = HEAD == 2 ? w2 : HEAD == 3 ? w3 : w0;
        uint32_t i;
        if (lean_reject(w, lcnt, i)) {
            odd = true;
        } else {
            const uint32_t e = pool[(uint64_t)linfo * LIST_UNIT_WORDS + i];
            v = pool[ls.adj + 2ull * e];
        }
    }
    if (odd) v = odd_step<MODE>(hdr, pool, u, seed, id, s, blk0, (uint32_t)TERM, rule);
    return v;
}

// ---------------------------------------------------------------------------
// Cooperative stepping: G lanes per walk.  With fewer walks than the chip has
// lanes a query's time is its longest chain of steps, and a step's time the
// loads it waits for one after the other.  The lanes of a walk therefore take
// apart what one lane does in turn: lane i computes block i of the step's stream
// (ahead, while the step before it waits for memory), so 4 G words are there at
// once; all member infos are loaded beside the header; and the first six or so
// dense attempts are loaded together.  A step waits for the header and one edge
// word (dense), or the header, a list entry and an edge word (listed).
// ---------------------------------------------------------------------------
template <int G>
struct CoopWords {
    uint32_t w[4];  // this lane's block (block `sub` of the step's stream)
    uint32_t z[4];  // block 0
};
template <int G>
__device__ __forceinline__ CoopWords<G> coop_words(uint64_t seed, uint64_t id, uint32_t s, uint32_t sub) {
    CoopWords<G> c;
    philox_uniform((uint32_t)id, (uint32_t)(id >> 32), s, sub, seed, c.w[0], c.w[1], c.w[2], c.w[3]);
    const int l0 = (int)(lane_id() - sub);
#pragma unroll
    for (int i = 0; i < 4; ++i) c.z[i] = __shfl(c.w[i], l0, 64);
    return c;
}

// One whole step at u of the walk that the G lanes share (act, u, id and s are
// the same in them; every lane of the wave calls).  Returns the next vertex or
// STOP_VERTEX in all G lanes.  mid() runs while the header loads are in flight.
template <int G, int MODE, int TERM, class Mid>
__device__ __forceinline__ uint32_t coop_step(const uint32_t* __restrict__ hdr, const uint32_t* __restrict__ pool,
                                              bool act, uint32_t u, uint64_t seed, uint64_t id, uint32_t s,
                                              const CoopWords<G>& cw, GroupRule rule, Mid mid) {
    constexpr uint32_t HEAD = TERM + (MODE == 2 ? 3 : 2);
    constexpr int IPL = G >= 32 ? 1 : 32 / G;  // infos per lane
    const uint32_t lane = lane_id(), sub = lane & (G - 1);
    const int l0 = (int)(lane - sub);
    uint32_t v = STOP_VERTEX;
    HotLine q;
    uint32_t inf[IPL] = {};
    if (act) {
        q = load_hot(hdr, u);
        const uint32_t* I = hdr_ref(hdr, u).cold + (H_INFO - HDR_HOT);
#pragma unroll
        for (int i = 0; i < IPL; ++i) inf[i] = G <= 32 || sub < 32 ? I[sub * IPL + i] : 0u;
    }
    const uint4 al = load_alias<MODE>(act, u, cw.z[TERM], rule);
    mid();
    LeanPick p;
    p.kind = LK_DONE;
    p.v = STOP_VERTEX;
    if (act)
        p = TERM ? lean_pick<MODE, WIDE_ODD>(hdr, u, q, cw.z[1], cw.z[2], cw.z[3], al, rule)
                 : lean_pick<MODE, WIDE_ODD>(hdr, u, q, cw.z[0], cw.z[1], cw.z[2], al, rule);
    // the list position's word, the list's offset
    uint32_t li = 0, info = 0;
    bool list = act && p.kind == LK_LIST;
    if (__ballot(list)) {
        const uint32_t w = HEAD < 4 ? cw.z[HEAD & 3] : __shfl(cw.w[0], l0 + 1, 64);
#pragma unroll
        for (int i = 0; i < IPL; ++i) {
            const uint32_t y = __shfl(inf[i], l0 + (int)(p.sel / IPL), 64);
            if (i == 0 || (p.sel % IPL) == (uint32_t)i) info = y;
        }
        if (list && lean_reject(w, p.csel, li)) {
            p.kind = LK_ODD;
            list = false;
        }
    }
    uint32_t le = 0;
    if (list) le = pool[(uint64_t)info * LIST_UNIT_WORDS + li];
    bool dense = act && p.kind == LK_DENSE;
    uint64_t dm = __ballot(dense);
    if (dm) {
        const uint64_t* __restrict__ edges = reinterpret_cast<const uint64_t*>(pool + p.adj);
#pragma unroll
        for (int round = 0; round < (G > 2 ? 2 : 1); ++round) {
            const bool mine = dense && (round == 0 ? sub < 2 : sub >= 2);
            uint64_t e[4];
            bool ok[4];
#pragma unroll
            for (int a = 0; a < 4; ++a) {
                uint32_t i;
                ok[a] = mine && !lean_reject(cw.w[a], p.d, i) && (sub > 0 || (uint32_t)a >= HEAD);
                e[a] = 0;
                if (ok[a]) e[a] = edges[i];
            }
            uint32_t got = PENDING;
#pragma unroll
            for (int a = 3; a >= 0; --a)
                if (ok[a] && (((uint32_t)(e[a] >> 32) >> p.sel) & 1u)) got = (uint32_t)e[a];
            const uint64_t am = group_bits<G>(__ballot(got != PENDING), (uint32_t)l0);
            const int src = am ? l0 + __ffsll((long long)am) - 1 : (int)lane;
            const uint32_t y = __shfl(got, src, 64);
            if (dense && am) {
                v = y;
                dense = false;
            }
            if (__ballot(dense) == 0) break;
        }
        if (dense) p.kind = LK_ODD;  // all the words at hand were rejected: again, one by one
        // The infos' registers stay theirs up to here: given to the attempts above while the loads are still under
        // way, they made an attempt's load wait for them (8 lanes, 30,000 PageRank walks 144 -> 152 us).
#pragma unroll
        for (int i = 0; i < IPL; ++i) asm volatile("" ::"v"(inf[i]));
    }
    if (list) v = pool[p.adj + 2ull * le];
    if (act && p.kind == LK_DONE) v = p.v;
    if (MODE == 1 && act && p.kind == LK_DEC)
        v = decimal_draw<HEAD>(hdr, pool, u, p, seed, id, s, 0u, cw.z[0], cw.z[1], cw.z[2], cw.z[3], rule);
    if (act && p.kind == LK_ODD) v = odd_step<MODE>(hdr, pool, u, seed, id, s, 0u, (uint32_t)TERM, rule);
    return v;
}

// The rest of a path after a vertex without out-edges, entries [from, L] of row,
// for every lane with `stop` set: written by the whole wave, 64 entries per
// store.  By its own lane alone it is a store of one word per entry (on an R-MAT
// graph more than half of all path entries are such padding).  Every lane of the
// wave must call this.
__device__ __forceinline__ void wave_pad_row(bool stop, uint32_t* row, uint32_t from, uint32_t L) {
    const uint32_t lane = lane_id();
    for (uint64_t m = __ballot(stop); m; m &= m - 1) {
        const int l = __ffsll((long long)m) - 1;
        const uint64_t r = ((uint64_t)__shfl((uint32_t)((uint64_t)row >> 32), l, 64) << 32) |
                           __shfl((uint32_t)(uint64_t)row, l, 64);
        uint32_t* p = reinterpret_cast<uint32_t*>(r);
        for (uint64_t x = (uint64_t)__shfl(from, l, 64) + lane; x <= L; x += 64) p[x] = STOP_VERTEX;  // L up to 2^32 - 2
    }
}

// Walk ids are handed to waves in chunks: one atomic per QCHUNK ids, and the
// lanes of a wave that need a walk take consecutive ids from the chunk.
struct WaveQueue {
    uint64_t next = 0, end = 0;  // identical in every lane of the wave
    uint32_t chunk = 256;
};

__device__ __forceinline__ uint64_t wave_take_chunked(bool need, WaveQueue& q, unsigned long long* head) {
    const uint64_t want = __ballot(need);
    if (!want) return NO_WALK;
    const uint32_t cnt = __popcll(want);
    const uint32_t rank = rank_below(want);
    const uint64_t avail = q.end - q.next;
    uint64_t id;
    if (avail >= cnt) {
        id = q.next + rank;
        q.next += cnt;
    } else {
        // reserve enough whole chunks for every lane that is still short
        const uint64_t chunks = (cnt - avail + q.chunk - 1) / q.chunk;
        unsigned long long nb = 0;
        if (lane_id() == 0) nb = atomicAdd(head, (unsigned long long)(chunks * q.chunk));
        nb = __shfl(nb, 0, 64);
        id = rank < avail ? q.next + rank : nb + (rank - avail);
        q.next = nb + (cnt - avail);
        q.end = nb + chunks * q.chunk;
    }
    return need ? id : NO_WALK;
}

__device__ __forceinline__ void wave_add_u64(unsigned long long* p, uint64_t v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    if (lane_id() == 0 && v) atomicAdd(p, (unsigned long long)v);
}
// The same with one atomic per block (every thread of the block calls): atomics on one word queue up at about 10 ns
// each, and short walks end in thousands of waves at once (30,000 walks of one step on eight lanes 52 us with one per
// wave, 18 now; 60,000 on a lane each 42 and 34).
template <int THREADS>
__device__ __forceinline__ void block_add_u64(unsigned long long* p, uint64_t v) {
    __shared__ uint64_t sh[THREADS / 64];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    if (lane_id() == 0) sh[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < THREADS / 64; ++w) v += sh[w];
        if (v) atomicAdd(p, (unsigned long long)v);
    }
}

}  // namespace
