// locate.hip -- building, sizing and checking the edge locator (locate.h).
// The batch pipeline (update.hip) keeps it in step with the adjacency; the
// streaming path marks it stale and the next batch that uses it rebuilds it.
#include "locate.h"
#include <stdio.h>
#include <algorithm>

namespace {

constexpr int WB = 256;

// every slot EMPTY, the chunk list behind them empty
__global__ void k_loc_clear(uint64_t* __restrict__ tab, uint64_t cap) {
    if (blockIdx.x == 0 && threadIdx.x == 0) tab[2 * cap] = 0;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < cap; i += (uint64_t)gridDim.x * blockDim.x)
        *reinterpret_cast<ulonglong2*>(tab + 2 * i) = make_ulonglong2(LOC_EMPTY, 0ull);
}

// Adds v over the block to *dst, one atomic per block: atomics on one word queue up at about 10 ns
// each, and one per wave of 16 M vertices cost more than the pass they ended.
__device__ __forceinline__ void block_sum_add(unsigned long long* dst, uint64_t v) {
    __shared__ uint64_t sh[WB / 64];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    __syncthreads();
    if (lane_id() == 0) sh[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (uint32_t w = 1; w < (blockDim.x >> 6); ++w) v += sh[w];
        if (v) atomicAdd(dst, (unsigned long long)v);
    }
}

// Building.  Every live edge claims a slot: a read and a write of one line at random, and the claims
// of different edges are independent, so what counts is how many are in flight.  A wave takes 64
// vertices, lane l the header of the l-th, and spreads their edges over its lanes, LB_EDGES claims in
// flight per lane; a vertex of more than LB_CHUNK edges goes to a list of chunks that a second launch
// works off, a block per chunk.  With a wave per vertex the largest hub set the time: 131 ms for 2^28
// edges of R-MAT 24, 39 ms for 2^24 with hubs of 3 x 10^5; now 30 ms and 3.1 ms, 9 x 10^9 and 5 x 10^9
// edges/s, bound by the lines at random.
constexpr uint32_t LB_CHUNK = 1024;
constexpr int LB_EDGES = 4;

// The chunk list lies behind the table's slots: its length, then (vertex << 32 | chunk).  A vertex of
// d > LB_CHUNK edges makes at most 2 d / LB_CHUNK entries, and the table has a slot per edge at least.
inline uint64_t chunk_list_words(uint64_t cap) { return 2 + 2 * cap / LB_CHUNK; }

// Claims for up to LB_EDGES edges per lane (key[j], index p[j], LOC_EMPTY: none); returns the failed
// ones.  The table was cleared and nothing is deleted meanwhile, so a slot is EMPTY or taken, and the
// compare-and-swap of the home slot needs no look at it first: at the loads kept here most succeed.
__device__ __forceinline__ uint32_t build_claims(const LocView& L, const uint64_t (&key)[LB_EDGES],
                                                 const uint32_t (&p)[LB_EDGES]) {
    uint64_t h[LB_EDGES], was[LB_EDGES];
#pragma unroll
    for (int j = 0; j < LB_EDGES; ++j) {
        h[j] = loc_hash(key[j]) & L.mask;
        was[j] = LOC_EMPTY;
        if (key[j] != LOC_EMPTY)
            was[j] = atomicCAS((unsigned long long*)(L.tab + 2 * h[j]), (unsigned long long)LOC_EMPTY,
                               (unsigned long long)key[j]);
    }
    uint32_t fail = 0;
#pragma unroll
    for (int j = 0; j < LB_EDGES; ++j) {
        const bool act = key[j] != LOC_EMPTY;
        if (act && was[j] == LOC_EMPTY) L.tab[2 * h[j] + 1] = p[j];
        uint32_t res = 1;
        uint64_t next = 0;
        if (act && was[j] != LOC_EMPTY) res = loc_claim_line(L, key[j], p[j], &next);
        loc_wave_claim(L, res == 0, key[j], p[j], next, &res);
        if (res == 0) ++fail;
    }
    return fail;
}

// cnt[0] += edges, cnt[1] += failed claims (of the vertices that do not go to the list)
__global__ void __launch_bounds__(WB) k_loc_build(const uint32_t* __restrict__ hdr, const uint32_t* __restrict__ pool,
                                                  uint32_t n, LocView L, unsigned long long* __restrict__ list,
                                                  unsigned long long* __restrict__ cnt) {
    const uint32_t lane = lane_id();
    uint64_t edges = 0;
    uint32_t fail = 0;
    const uint64_t step = (uint64_t)gridDim.x * WB;
    for (uint64_t u0 = (uint64_t)blockIdx.x * WB + (threadIdx.x & ~63u); u0 < n; u0 += step) {
        const uint64_t u = u0 + lane;
        uint32_t d = 0;
        uint64_t adj = 0;
        if (u < n) {
            const HdrCRef h = hdr_ref(hdr, u);
            d = h[H_DEG];
            adj = hdr_adj(h);
        }
        edges += d;
        const uint32_t ch = d > LB_CHUNK ? (d + LB_CHUNK - 1) / LB_CHUNK : 0;
        uint32_t x = ch, y = ch ? 0 : d;  // inclusive sums over the lanes
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t xx = __shfl_up(x, o, 64), yy = __shfl_up(y, o, 64);
            if (lane >= (uint32_t)o) {
                x += xx;
                y += yy;
            }
        }
        if (__shfl(x, 63, 64)) {
            unsigned long long at = 0;
            if (lane == 63) at = atomicAdd(list, (unsigned long long)x);
            at = __shfl(at, 63, 64) + x - ch;
            for (uint32_t c = 0; c < ch; ++c) list[1 + at + c] = (u << 32) | c;
        }
        const uint32_t total = __shfl(y, 63, 64);
        const uint32_t y0 = y - (ch ? 0 : d);
        for (uint32_t e0 = 0; e0 < total; e0 += 64 * LB_EDGES) {
            uint64_t key[LB_EDGES];
            uint32_t p[LB_EDGES];
#pragma unroll
            for (int j = 0; j < LB_EDGES; ++j) {
                const uint32_t e = e0 + 64 * j + lane;
                // the first lane whose inclusive sum is past e
                uint32_t o = 0;
#pragma unroll
                for (int s = 32; s > 0; s >>= 1)
                    if (__shfl(y, (int)(o + s - 1), 64) <= e) o += s;
                o &= 63;  // e past the total
                p[j] = e - __shfl(y0, (int)o, 64);
                const uint64_t a = __shfl(adj, (int)o, 64);
                key[j] = e < total ? loc_key((uint32_t)u0 + o, pool[a + 2ull * p[j]]) : LOC_EMPTY;
            }
            fail += build_claims(L, key, p);
        }
    }
    block_sum_add(cnt, edges);
    block_sum_add(cnt + 1, fail);
}

// the listed chunks; cnt[1] += failed claims
__global__ void __launch_bounds__(WB) k_loc_build_chunks(const uint32_t* __restrict__ hdr,
                                                         const uint32_t* __restrict__ pool, LocView L,
                                                         const unsigned long long* __restrict__ list,
                                                         unsigned long long* __restrict__ cnt) {
    static_assert(LB_CHUNK % (WB * LB_EDGES) == 0, "whole rounds");
    uint32_t fail = 0;
    const uint64_t items = list[0];
    for (uint64_t i = blockIdx.x; i < items; i += gridDim.x) {
        const uint32_t u = (uint32_t)(list[1 + i] >> 32), c = (uint32_t)list[1 + i];
        const HdrCRef h = hdr_ref(hdr, u);
        const uint32_t d = h[H_DEG], to = min(d, (c + 1) * LB_CHUNK);
        const uint64_t adj = hdr_adj(h);
        for (uint32_t e0 = c * LB_CHUNK; e0 < to; e0 += WB * LB_EDGES) {
            uint64_t key[LB_EDGES];
            uint32_t p[LB_EDGES];
#pragma unroll
            for (int j = 0; j < LB_EDGES; ++j) {
                p[j] = e0 + WB * j + threadIdx.x;
                key[j] = p[j] < to ? loc_key(u, pool[adj + 2ull * p[j]]) : LOC_EMPTY;
            }
            fail += build_claims(L, key, p);
        }
    }
    block_sum_add(cnt + 1, fail);
}

// Consistency: every live edge finds its own slot (cnt[0] counts those that do not),
// and the table holds no other live slot (cnt[1] counts live slots).
__global__ void __launch_bounds__(WB) k_loc_check_edges(const uint32_t* __restrict__ hdr,
                                                        const uint32_t* __restrict__ pool, uint32_t n, LocView L,
                                                        unsigned long long* __restrict__ cnt) {
    const uint32_t lane = lane_id();
    uint32_t bad = 0;
    for (uint64_t u = (uint64_t)blockIdx.x * (WB / 64) + (threadIdx.x >> 6); u < n; u += (uint64_t)gridDim.x * (WB / 64)) {
        const HdrCRef h = hdr_ref(hdr, u);
        const uint32_t d = h[H_DEG];
        const uint64_t adj = hdr_adj(h);
        for (uint32_t i = lane; i < d; i += 64)
            if (loc_find(L, loc_key((uint32_t)u, pool[adj + 2ull * i]), i) == LOC_EMPTY) ++bad;
    }
    bad = loc_wave_sum(bad);
    if (lane == 0 && bad) atomicAdd(cnt, (unsigned long long)bad);
}

__global__ void k_loc_count_live(LocView L, unsigned long long* __restrict__ cnt) {
    uint32_t live = 0;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i <= L.mask; i += (uint64_t)gridDim.x * blockDim.x) {
        const uint64_t k = L.tab[2 * i];
        if (k != LOC_EMPTY && k != LOC_TOMB) ++live;
    }
    live = loc_wave_sum(live);
    if (lane_id() == 0 && live) atomicAdd(cnt + 1, (unsigned long long)live);
}

uint32_t grid_of(uint64_t items, uint32_t per_block) {
    return (uint32_t)std::max<uint64_t>(1, std::min<uint64_t>((items + per_block - 1) / per_block, 1u << 16));
}

// blocks of the building passes: 32 waves on each of 256 compute units
constexpr uint32_t LB_GRID = 2048;

// Rebuild into a table of `cap` slots (reallocated when the capacity changes).
bool loc_build(bingo_graph* g, uint64_t cap, hipStream_t st) {
    g->loc_valid = false;
    if (cap != g->loc_cap || !g->loc_tab) {
        // the captured update graphs hold the old table's address
        update_drop_graphs(g);
        hipFree(g->loc_tab);
        g->loc_tab = nullptr;
        g->loc_cap = 0;
        if (dev_malloc(&g->loc_tab, (2 * cap + chunk_list_words(cap)) * 8) != hipSuccess) {
            (void)hipGetLastError();
            g->loc_tab = nullptr;
            return false;
        }
        g->loc_cap = cap;
    }
    const LocView L{g->loc_tab, cap - 1};
    unsigned long long* cnt = g->d_ctl + CTL_LOC;
    if (hipMemsetAsync(cnt, 0, 16, st) != hipSuccess) return false;
    hipLaunchKernelGGL(k_loc_clear, dim3(grid_of(cap, 256)), dim3(256), 0, st, g->loc_tab, cap);
    unsigned long long* list = (unsigned long long*)(g->loc_tab + 2 * cap);
    hipLaunchKernelGGL(k_loc_build, dim3(std::min(grid_of(g->n, WB), LB_GRID)), dim3(WB), 0, st,
                       (const uint32_t*)g->hdr, (const uint32_t*)g->pool, g->n, L, list, cnt);
    hipLaunchKernelGGL(k_loc_build_chunks, dim3(std::min(grid_of(cap, LB_CHUNK), LB_GRID)), dim3(WB), 0, st,
                       (const uint32_t*)g->hdr, (const uint32_t*)g->pool, L, (const unsigned long long*)list, cnt);
    unsigned long long c[2] = {0, 0};
    if (hipMemcpyAsync(c, cnt, 16, hipMemcpyDeviceToHost, st) != hipSuccess || hipStreamSynchronize(st) != hipSuccess)
        return false;
    if (c[1]) return false;  // unreachable: the capacity is at least 1.6 times the edges
    g->loc_live = g->loc_used = c[0];
    g->loc_valid = true;
    return true;
}

uint64_t pow2_ge(uint64_t x) {
    uint64_t c = 1ull << 16;
    while (c < x) c <<= 1;
    return c;
}

// live edges of the structure (one pass over the headers)
__global__ void __launch_bounds__(WB) k_loc_edges(const uint32_t* __restrict__ hdr, uint32_t n,
                                                  unsigned long long* __restrict__ cnt) {
    uint64_t s = 0;
    for (uint64_t u = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; u < n; u += (uint64_t)gridDim.x * blockDim.x)
        s += hdr_ref(hdr, u)[H_DEG];
    block_sum_add(cnt, s);
}

}  // namespace

LocView locator_view(const bingo_graph* g) {
    if (!g->update_locate || !g->loc_valid) return LocView{nullptr, 0};
    return LocView{g->loc_tab, g->loc_cap - 1};
}

bool locator_prepare(bingo_graph* g, uint64_t n_ins, hipStream_t st) {
    if (!g->update_locate || g->radix_base != 2) return false;
    // load limits: at most 0.8 of the slots taken (live + TOMB) after the batch's claims; a
    // rebuild sizes the table to at least 1.6 times the live edges plus the batch
    if (g->loc_valid && (double)(g->loc_used + n_ins) <= 0.8 * (double)g->loc_cap) return true;
    uint64_t live = g->loc_live;
    if (!g->loc_valid) {
        unsigned long long* cnt = g->d_ctl + CTL_LOC;
        unsigned long long c = 0;
        if (hipMemsetAsync(cnt, 0, 8, st) != hipSuccess) return false;
        hipLaunchKernelGGL(k_loc_edges, dim3(std::min(grid_of(g->n, WB), LB_GRID)), dim3(WB), 0, st, (const uint32_t*)g->hdr, g->n, cnt);
        if (hipMemcpyAsync(&c, cnt, 8, hipMemcpyDeviceToHost, st) != hipSuccess ||
            hipStreamSynchronize(st) != hipSuccess)
            return false;
        live = c;
    }
    const uint64_t want = pow2_ge((uint64_t)(1.6 * (double)(live + n_ins)) + 1);
    // keep a larger table that still fits the limit rather than shrinking it
    const uint64_t cap = (g->loc_cap >= want && (double)(live + n_ins) <= 0.5 * (double)g->loc_cap) ? g->loc_cap : want;
    return loc_build(g, cap, st);
}

void locator_after_batch(bingo_graph* g, uint64_t kills, uint64_t claims, uint64_t fresh, uint64_t bad) {
    if (!g->loc_valid) return;
    if (bad) {
        fprintf(stderr, "libbingo: edge locator out of step (%llu lookups failed); it will be rebuilt\n",
                (unsigned long long)bad);
        g->loc_valid = false;
        return;
    }
    g->loc_live = g->loc_live + claims - kills;
    g->loc_used += fresh;
}

void locator_invalidate(bingo_graph* g) { g->loc_valid = false; }

void locator_release(bingo_graph* g) {
    hipFree(g->loc_tab);
    g->loc_tab = nullptr;
    g->loc_cap = g->loc_live = g->loc_used = 0;
    g->loc_valid = false;
}

extern "C" int bingo_check_locator(bingo_graph* g, uint64_t* h_bad, uint64_t* h_live, void* stream) {
    if (!g || !h_bad || g->radix_base != 2) return BINGO_E_INVALID;
    if (!g->loc_valid) return BINGO_E_INVALID;
    hipStream_t st = (hipStream_t)stream;
    const LocView L{g->loc_tab, g->loc_cap - 1};
    unsigned long long* cnt = g->d_ctl + CTL_LOC;
    HIPCHK(hipMemsetAsync(cnt, 0, 16, st));
    hipLaunchKernelGGL(k_loc_check_edges, dim3(grid_of(g->n, WB / 64)), dim3(WB), 0, st, (const uint32_t*)g->hdr,
                       (const uint32_t*)g->pool, g->n, L, cnt);
    hipLaunchKernelGGL(k_loc_count_live, dim3(grid_of(g->loc_cap, 256)), dim3(256), 0, st, L, cnt);
    unsigned long long c[2] = {0, 0};
    HIPCHK(hipMemcpyAsync(c, cnt, 16, hipMemcpyDeviceToHost, st));
    HIPCHK(hipStreamSynchronize(st));
    // edges without their slot, plus live slots beyond the edges (or edges beyond the live slots)
    unsigned long long edges = 0;
    {
        HIPCHK(hipMemsetAsync(cnt, 0, 8, st));
        hipLaunchKernelGGL(k_loc_edges, dim3(std::min(grid_of(g->n, WB), LB_GRID)), dim3(WB), 0, st, (const uint32_t*)g->hdr, g->n, cnt);
        HIPCHK(hipMemcpyAsync(&edges, cnt, 8, hipMemcpyDeviceToHost, st));
        HIPCHK(hipStreamSynchronize(st));
    }
    *h_bad = c[0] + (c[1] > edges ? c[1] - edges : edges - c[1]) + (c[1] != g->loc_live ? 1 : 0);
    if (h_live) *h_live = c[1];
    return BINGO_OK;
}
