// api.hip -- the extern "C" entry points of libbingo (declared in bingo.h).
#include "dev.h"
#include "locate.h"
#include <stdio.h>
#include <string.h>
#include <new>
#include <stdlib.h>
#include <cmath>
#include <mutex>
#include <unordered_map>
#include <vector>

// ---------------------------------------------------------------------------
// Large blocks between graphs.  The driver clears freed device memory before it
// hands it out again, at about 25 GB/s once the memory that was clean from the
// start is used up, so a program that builds and destroys graphs in turn waits for
// that: 77 ms per graph of 2^20 vertices and 2^24 edges (2 GB in all), whose build
// takes 3 ms of device time.  A destroyed graph's headers, pool and workspace
// are therefore kept for the next one: at most DEV_KEEP bytes in the process, a
// block of at most a quarter more than is asked for, and not for longer than
// DEV_AGE later frees; bingo_trim gives them all back, and so does every device
// allocation of the library that fails, which is then tried once more.  Blocks
// under 1 MiB are not kept.  A block belongs to the device that was current at
// its allocation, and is kept only by calls that have waited for that device.
// ---------------------------------------------------------------------------
namespace {
constexpr size_t DEV_KEEP = 4ull << 30;
constexpr size_t DEV_LEAST = 1ull << 20;
constexpr uint64_t DEV_AGE = 32;
struct DevBlock {
    void* p;
    size_t bytes;
    int dev;
    uint64_t tick;
};
struct DevBlocks {
    std::mutex mu;
    std::vector<DevBlock> idle;                // in order of freeing
    std::unordered_map<void*, DevBlock> live;  // blocks in use that may be kept
    size_t idle_bytes = 0;
    uint64_t tick = 0;
    // give back idle blocks, all or those past the bounds; returns their bytes
    size_t trim(bool all) {
        size_t keep = 0, given = 0;
        for (size_t i = 0; i < idle.size(); ++i) {
            DevBlock& b = idle[i];
            // the oldest come first
            if (all || idle_bytes > DEV_KEEP || tick - b.tick > DEV_AGE) {
                hipFree(b.p);
                idle_bytes -= b.bytes;
                given += b.bytes;
            } else {
                idle[keep++] = b;
            }
        }
        idle.resize(keep);
        return given;
    }
};
DevBlocks& dev_blocks() {
    static DevBlocks* b = new DevBlocks();  // never destroyed: the process's end gives the memory back
    return *b;
}
// sizes in steps of an eighth of their power of two, so that graphs of about one size share blocks
size_t dev_round(size_t bytes) {
    size_t step = 1ull << 17;
    while ((step << 4) <= bytes) step <<= 1;
    return (bytes + step - 1) & ~(step - 1);
}
// `get` until it succeeds, at most twice: the idle blocks are given back in between
template <class F>
hipError_t dev_try(F get) {
    hipError_t e = get();
    if (e == hipSuccess) return e;
    (void)hipGetLastError();
    if (!dev_trim()) return e;
    e = get();
    if (e != hipSuccess) (void)hipGetLastError();
    return e;
}
}  // namespace

size_t dev_trim() {
    DevBlocks& d = dev_blocks();
    std::lock_guard<std::mutex> lk(d.mu);
    return d.trim(true);
}

hipError_t dev_malloc(void** p, size_t bytes) {
    const hipError_t e = dev_try([&] { return hipMalloc(p, bytes); });
    if (e != hipSuccess) *p = nullptr;
    return e;
}

hipError_t dev_malloc_async(void** p, size_t bytes, hipStream_t st) {
    const hipError_t e = dev_try([&] { return hipMallocAsync(p, bytes, st); });
    if (e != hipSuccess) *p = nullptr;
    return e;
}

void* dev_alloc(size_t bytes) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return nullptr;
    // what is never kept is not rounded up either
    const bool keep = bytes >= DEV_LEAST && dev_round(bytes) <= DEV_KEEP;
    void* p = nullptr;
    if (!keep) return dev_malloc(&p, bytes) == hipSuccess ? p : nullptr;
    DevBlocks& d = dev_blocks();
    size_t want = dev_round(bytes);
    try {
        std::lock_guard<std::mutex> lk(d.mu);
        size_t best = d.idle.size();
        for (size_t i = 0; i < d.idle.size(); ++i) {
            const DevBlock& b = d.idle[i];
            if (b.dev == dev && b.bytes >= want && b.bytes <= want + want / 4 &&
                (best == d.idle.size() || b.bytes < d.idle[best].bytes))
                best = i;
        }
        if (best < d.idle.size()) {
            const DevBlock b = d.idle[best];
            d.live[b.p] = b;
            d.idle.erase(d.idle.begin() + (long)best);
            d.idle_bytes -= b.bytes;
            return b.p;
        }
    } catch (const std::bad_alloc&) {
        // no host memory for the list's entry: the block stays idle
    }
    if (hipMalloc(&p, want) != hipSuccess) {
        (void)hipGetLastError();
        want = bytes;  // near the end of the memory: the exact size
        if (dev_malloc(&p, want) != hipSuccess) return nullptr;
    }
    try {
        std::lock_guard<std::mutex> lk(d.mu);
        d.live[p] = DevBlock{p, want, dev, 0};
    } catch (const std::bad_alloc&) {
        // not listed: dev_free gives it back instead of keeping it
    }
    return p;
}

void dev_free(void* p, bool idle) {
    if (!p) return;
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess) dev = -1;
    DevBlocks& d = dev_blocks();
    std::lock_guard<std::mutex> lk(d.mu);
    const auto it = d.live.find(p);
    bool kept = false;
    if (it != d.live.end()) {
        DevBlock b = it->second;
        d.live.erase(it);
        if (idle && b.dev == dev) {
            b.tick = d.tick;
            try {
                d.idle.push_back(b);
                d.idle_bytes += b.bytes;
                kept = true;
            } catch (const std::bad_alloc&) {
            }
        }
    }
    if (!kept) hipFree(p);
    ++d.tick;
    d.trim(false);
}

void* ws_get(bingo_graph* g, size_t bytes) {
    // a pending asynchronous PPR histogram still reads its visit bins here
    if (ppr_drain(g) != BINGO_OK) return nullptr;
    if (bytes <= g->ws_bytes && g->ws) return g->ws;
    dev_free(g->ws, hipDeviceSynchronize() == hipSuccess);
    g->ws = nullptr;
    g->ws_bytes = 0;
    const size_t want = bytes + bytes / 4 + 4096;
    g->ws = dev_alloc(want);
    if (!g->ws) return nullptr;
    g->ws_bytes = want;
    return g->ws;
}

// Record the next phase boundary of the current call on its stream.
void phase_mark(bingo_graph* g, hipStream_t st, bool first) {
    if (first) g->nev = 0;
    if (g->nev >= PHASE_EVENTS) return;
    if (!g->ev[g->nev] && hipEventCreate(&g->ev[g->nev]) != hipSuccess) return;
    if (hipEventRecord(g->ev[g->nev], st) == hipSuccess) g->nev++;
}

int err_to_code(uint32_t bits) {
    if (bits & ERR_RANGE) return BINGO_E_RANGE;
    if (bits & ERR_WEIGHT) return BINGO_E_WEIGHT;
    if (bits & ERR_OOM) return BINGO_E_OOM;
    if (bits & ERR_INTERNAL) return BINGO_E_INTERNAL;
    return BINGO_OK;
}

// Free everything the handle owns; idle: the current device has finished all work on it.
static void release(bingo_graph* g, bool idle) {
    if (!g) return;
    update_release(g);
    locator_release(g);
    for (int i = 0; i < PHASE_EVENTS; ++i)
        if (g->ev[i]) hipEventDestroy(g->ev[i]);
    for (int i = 0; i < WALK_SLOTS; ++i)
        if (g->slot_ev[i]) hipEventDestroy(g->slot_ev[i]);
    for (hipEvent_t e : {g->ppr_done, g->ppr_h0, g->ppr_h1})
        if (e) hipEventDestroy(e);
    dev_free(g->hdr_mem, idle);
    hipFree(g->alias);
    dev_free(g->pool, idle);
    hipFree(g->d_ctl);
    hipFree(g->d_err);
    hipFree(g->ppr_off);
    hipFree(g->ppr_vtx);
    hipFree(g->ppr_cnt);
    dev_free(g->ws, idle);
    hipFree(g->aux);
    hipFree(g->n2v_idx);
    hipFree(g->n2v_off);
    delete g;
}

extern "C" {

int bingo_build(const bingo_config* cfg, uint32_t n, uint64_t m, const uint32_t* d_src, const uint32_t* d_dst,
                const uint32_t* d_w, void* stream, bingo_graph** out) {
    if (!out) return BINGO_E_INVALID;
    *out = nullptr;
    if (!cfg || cfg->struct_size != sizeof(bingo_config)) return BINGO_E_INVALID;
    if (n == 0 || n >= (1u << 31) || m >= (1ull << 32)) return BINGO_E_INVALID;
    if (m && (!d_src || !d_dst || !d_w)) return BINGO_E_INVALID;
    if (cfg->adaptive > 1 || cfg->alpha_pct > 100 || cfg->beta_pct > 100) return BINGO_E_INVALID;
    if (cfg->frac_bits > 16 || cfg->alias_table > 1 || (cfg->alias_table && cfg->frac_bits)) return BINGO_E_INVALID;
    const uint32_t radix = cfg->radix_base ? cfg->radix_base : 2u;
    if ((radix != 2 && radix != 4) || cfg->reserved) return BINGO_E_INVALID;
    if (radix == 4 && (cfg->frac_bits || cfg->alias_table)) return BINGO_E_INVALID;
    hipStream_t st = (hipStream_t)stream;
    bingo_graph* g = new (std::nothrow) bingo_graph();
    if (!g) return BINGO_E_OOM;
    g->n = n;
    g->rule.adaptive = cfg->adaptive;
    g->rule.alpha = cfg->alpha_pct;
    g->rule.beta = cfg->beta_pct;
    g->rule.fbits = cfg->frac_bits;
    g->rule.alias = nullptr;
    g->alias_mode = cfg->alias_table;
    g->pool_words = cfg->pool_bytes / 4;
    g->pool_auto = cfg->pool_bytes == 0;
    g->radix_base = radix;
    const uint64_t hdr_words = radix == 4 ? (uint64_t)n * H4_WORDS : hdr_total_words(n);
    g->hdr = g->hdr_mem = nullptr; g->pool = nullptr; g->d_ctl = nullptr; g->d_err = nullptr; g->alias = nullptr;
    if (!(g->hdr_mem = (uint32_t*)dev_alloc(hdr_words * 4)) ||
        dev_malloc(&g->d_ctl, CTL_WORDS * 8) != hipSuccess || dev_malloc(&g->d_err, 4) != hipSuccess) {
        release(g, true);
        return BINGO_E_OOM;
    }
    g->hdr = radix == 4 ? g->hdr_mem : g->hdr_mem + hdr_front_words(n);
    if (hipMemsetAsync(g->hdr_mem, 0, hdr_words * 4, st) != hipSuccess ||
        hipMemsetAsync(g->d_ctl, 0, CTL_WORDS * 8, st) != hipSuccess) {
        release(g, hipStreamSynchronize(st) == hipSuccess);
        return BINGO_E_HIP;
    }
    const int rc = build_graph(g, m, d_src, d_dst, d_w, st);
    if (rc != BINGO_OK) {
        release(g, hipStreamSynchronize(st) == hipSuccess);
        return rc;
    }
    *out = g;
    return BINGO_OK;
}

int bingo_quantize_biases(uint64_t m, const float* d_bias, double lambda, uint32_t frac_bits, uint32_t* d_w,
                          void* stream) {
    if (m && (!d_bias || !d_w)) return BINGO_E_INVALID;
    if (frac_bits < 1 || frac_bits > 16 || !(lambda > 0.0) || std::isinf(lambda)) return BINGO_E_INVALID;
    return quantize_biases(m, d_bias, lambda, frac_bits, d_w, (hipStream_t)stream);
}

int bingo_update_batch(bingo_graph* g, uint64_t n_ins, const uint32_t* d_ins_src, const uint32_t* d_ins_dst,
                       const uint32_t* d_ins_w, uint64_t n_del, const uint32_t* d_del_src, const uint32_t* d_del_dst,
                       void* stream, bingo_update_stats* h_stats) {
    if (!g || g->radix_base != 2) return BINGO_E_INVALID;
    if (n_ins && (!d_ins_src || !d_ins_dst || !d_ins_w)) return BINGO_E_INVALID;
    if (n_del && (!d_del_src || !d_del_dst)) return BINGO_E_INVALID;
    return update_batch(g, n_ins, d_ins_src, d_ins_dst, d_ins_w, n_del, d_del_src, d_del_dst, h_stats,
                        (hipStream_t)stream);
}

int bingo_update_stream(bingo_graph* g, uint64_t n, const uint32_t* d_op, const uint32_t* d_src,
                        const uint32_t* d_dst, const uint32_t* d_w, void* stream, bingo_update_stats* h_stats) {
    if (!g || g->radix_base != 2 || (n && (!d_op || !d_src || !d_dst || !d_w))) return BINGO_E_INVALID;
    return update_stream(g, n, d_op, d_src, d_dst, d_w, h_stats, (hipStream_t)stream);
}

int bingo_walk(const bingo_graph* g, uint64_t n_walks, const uint32_t* d_starts, uint64_t walk_id_base,
               uint32_t length, uint64_t seed, uint32_t* d_paths, uint64_t* d_steps_taken, uint32_t mode,
               void* stream) {
    if (!g || (n_walks && (!d_starts || !d_paths))) return BINGO_E_INVALID;
    if (mode > BINGO_WALK_PER_STEP || length == 0xFFFFFFFFu) return BINGO_E_INVALID;
    if (g->radix_base == 4) {
        if (mode != BINGO_WALK_PERSISTENT) return BINGO_E_INVALID;
        return launch_walk4(const_cast<bingo_graph*>(g), n_walks, d_starts, walk_id_base, length, seed, d_paths,
                            d_steps_taken, (hipStream_t)stream);
    }
    return launch_walk(const_cast<bingo_graph*>(g), n_walks, d_starts, walk_id_base, length, seed, d_paths,
                       d_steps_taken, mode, (hipStream_t)stream);
}

int bingo_walk_batch(const bingo_graph* g, uint32_t n_queries, const bingo_walk_query* h_queries, void* stream) {
    if (!g || g->radix_base != 2 || n_queries > BINGO_WALK_BATCH_MAX || (n_queries && !h_queries)) return BINGO_E_INVALID;
    for (uint32_t i = 0; i < n_queries; ++i) {
        const bingo_walk_query& q = h_queries[i];
        if ((q.n_walks && (!q.d_starts || !q.d_paths)) || q.length == 0xFFFFFFFFu) return BINGO_E_INVALID;
    }
    return launch_walk_batch(const_cast<bingo_graph*>(g), n_queries, h_queries, (hipStream_t)stream);
}

int bingo_node2vec(bingo_graph* g, uint64_t n_walks, const uint32_t* d_starts, uint64_t walk_id_base,
                   uint32_t length, double p, double q, uint64_t seed, uint32_t* d_paths, uint64_t* d_counts,
                   void* stream) {
    if (!g || g->radix_base != 2 || (n_walks && (!d_starts || !d_paths)) || length == 0xFFFFFFFFu)
        return BINGO_E_INVALID;
    return run_node2vec(g, n_walks, d_starts, walk_id_base, length, p, q, seed, d_paths, d_counts,
                        (hipStream_t)stream);
}

int bingo_ppr(bingo_graph* g, uint32_t n_sources, const uint32_t* d_sources, uint32_t walks_per_source,
              uint32_t term_threshold, uint32_t max_len, uint64_t seed, uint64_t walk_id_base, uint32_t mode,
              uint64_t* h_total_entries, uint64_t* h_total_steps, void* stream) {
    if (!g || g->radix_base != 2 || !h_total_entries || n_sources == 0 || walks_per_source == 0 || !d_sources)
        return BINGO_E_INVALID;
    if (mode > BINGO_WALK_PER_STEP) return BINGO_E_INVALID;
    if ((uint64_t)n_sources * walks_per_source >= (1ull << 40)) return BINGO_E_INVALID;
    return run_ppr(g, n_sources, d_sources, walks_per_source, term_threshold, max_len, seed, walk_id_base, mode,
                   h_total_entries, h_total_steps, (hipStream_t)stream);
}

int bingo_ppr_async(bingo_graph* g, uint32_t n_sources, const uint32_t* d_sources, uint32_t walks_per_source,
                    uint32_t term_threshold, uint32_t max_len, uint64_t seed, uint64_t walk_id_base,
                    uint64_t* h_total_steps, void* stream, void* hist_stream) {
    if (!g || g->radix_base != 2 || n_sources == 0 || walks_per_source == 0 || !d_sources) return BINGO_E_INVALID;
    if ((uint64_t)n_sources * walks_per_source >= (1ull << 40)) return BINGO_E_INVALID;
    uint64_t entries = 0;
    return run_ppr(g, n_sources, d_sources, walks_per_source, term_threshold, max_len, seed, walk_id_base,
                   BINGO_WALK_PERSISTENT, &entries, h_total_steps, (hipStream_t)stream, (hipStream_t)hist_stream);
}

int bingo_ppr_wait(bingo_graph* g, uint64_t* h_total_entries, float* h_hist_ms) {
    if (!g) return BINGO_E_INVALID;
    return ppr_wait(g, h_total_entries, h_hist_ms);
}

int bingo_ppr_fetch(bingo_graph* g, uint64_t* d_offsets, uint32_t* d_vertex, uint32_t* d_count, uint64_t capacity,
                    void* stream) {
    if (!g || !d_offsets || !d_vertex || !d_count || !g->ppr_off) return BINGO_E_INVALID;
    if (int rc = ppr_drain(g)) return rc;
    if (capacity < g->ppr_entries) return BINGO_E_CAPACITY;
    hipStream_t st = (hipStream_t)stream;
    HIPCHK(hipMemcpyAsync(d_offsets, g->ppr_off, ((uint64_t)g->ppr_nsrc + 1) * 8, hipMemcpyDeviceToDevice, st));
    if (g->ppr_entries) {
        HIPCHK(hipMemcpyAsync(d_vertex, g->ppr_vtx, g->ppr_entries * 4, hipMemcpyDeviceToDevice, st));
        HIPCHK(hipMemcpyAsync(d_count, g->ppr_cnt, g->ppr_entries * 4, hipMemcpyDeviceToDevice, st));
    }
    return BINGO_OK;
}

int bingo_export(bingo_graph* g, uint32_t* h_buf, uint64_t cap_words, uint64_t* h_len, void* stream) {
    if (!g || !h_len) return BINGO_E_INVALID;
    if (int rc = ppr_drain(g)) return rc;
    if (g->radix_base == 4) return export_graph4(g, 0, g->n, h_buf, cap_words, h_len, (hipStream_t)stream);
    return export_graph(g, 0, g->n, h_buf, cap_words, h_len, (hipStream_t)stream);
}

int bingo_export_range(bingo_graph* g, uint32_t u_begin, uint32_t u_end, uint32_t* h_buf, uint64_t cap_words,
                       uint64_t* h_len, void* stream) {
    if (!g || !h_len) return BINGO_E_INVALID;
    if (int rc = ppr_drain(g)) return rc;
    if (g->radix_base == 4) return export_graph4(g, u_begin, u_end, h_buf, cap_words, h_len, (hipStream_t)stream);
    return export_graph(g, u_begin, u_end, h_buf, cap_words, h_len, (hipStream_t)stream);
}

int bingo_export_index_range(bingo_graph* g, uint32_t u_begin, uint32_t u_end, uint32_t* h_buf, uint64_t cap_words,
                             uint64_t* h_len, void* stream) {
    if (!g || !h_len || g->radix_base != 2) return BINGO_E_INVALID;
    if (int rc = ppr_drain(g)) return rc;
    return export_index(g, u_begin, u_end, h_buf, cap_words, h_len, (hipStream_t)stream);
}

int bingo_compact(bingo_graph* g, uint64_t pool_bytes, void* stream) {
    if (!g || g->radix_base != 2) return BINGO_E_INVALID;
    if (int rc = ppr_drain(g)) return rc;
    if (pool_bytes > (1ull << 37)) return BINGO_E_INVALID;
    return compact_pool(g, pool_bytes / 4, (hipStream_t)stream);
}

int bingo_memory(bingo_graph* g, bingo_mem_stats* out, void* stream) {
    if (!g || !out) return BINGO_E_INVALID;
    if (int rc = ppr_drain(g)) return rc;
    memset(out, 0, sizeof(*out));
    if (g->radix_base == 4) return memory_stats4(g, out, (hipStream_t)stream);
    return memory_stats(g, out, (hipStream_t)stream);
}

int bingo_status(bingo_graph* g, void* stream) {
    if (!g) return BINGO_E_INVALID;
    if (int rc = ppr_drain(g)) return rc;
    hipStream_t st = (hipStream_t)stream;
    uint32_t bits = 0;
    HIPCHK(hipMemcpyAsync(&bits, g->d_err, 4, hipMemcpyDeviceToHost, st));
    HIPCHK(hipStreamSynchronize(st));
    HIPCHK(hipMemsetAsync(g->d_err, 0, 4, st));
    return err_to_code(bits);
}

uint32_t bingo_num_vertices(const bingo_graph* g) { return g ? g->n : 0u; }

int bingo_set_tuning(bingo_graph* g, const bingo_tuning* t) {
    if (!g || !t || t->struct_size != sizeof(bingo_tuning)) return BINGO_E_INVALID;
    if (t->walk_variant > 1 || t->blocks_per_cu > 64 || t->update_graphs > 1 || t->ppr_bins > 1 ||
        t->update_locate > 1)
        return BINGO_E_INVALID;
    if (t->update_split != 0 && t->update_split < 64) return BINGO_E_INVALID;
    const uint32_t qc = t->queue_chunk ? t->queue_chunk : 256u;
    if (qc < 16 || qc > 4096 || (qc & (qc - 1))) return BINGO_E_INVALID;
    const uint32_t ds = t->dense_spec ? t->dense_spec : 2u;
    if (ds != 1 && ds != 2 && ds != 4) return BINGO_E_INVALID;
    g->dense_spec = ds;
    g->ppr_bins = t->ppr_bins;
    g->update_split = t->update_split;
    g->walk_variant = t->walk_variant;
    g->blocks_per_cu = t->blocks_per_cu;
    g->queue_chunk = qc;
    g->update_graphs = t->update_graphs;
    g->wave_degree = t->wave_degree;
    g->update_locate = t->update_locate;
    return BINGO_OK;
}

int bingo_get_tuning(const bingo_graph* g, bingo_tuning* t) {
    if (!g || !t) return BINGO_E_INVALID;
    t->struct_size = sizeof(bingo_tuning);
    t->walk_variant = g->walk_variant;
    t->blocks_per_cu = g->blocks_per_cu;
    t->queue_chunk = g->queue_chunk;
    t->update_graphs = g->update_graphs;
    t->dense_spec = g->dense_spec;
    t->ppr_bins = g->ppr_bins;
    t->update_split = g->update_split;
    t->wave_degree = g->wave_degree;
    t->update_locate = g->update_locate;
    return BINGO_OK;
}

int bingo_last_phase_ms(bingo_graph* g, float* h_ms, uint32_t cap, uint32_t* h_n) {
    if (!g || !h_n) return BINGO_E_INVALID;  // a pending histogram records no phase: no wait
    const uint32_t n = g->nev > 1 ? g->nev - 1 : 0;
    *h_n = n;
    if (!h_ms) return BINGO_OK;
    if (cap < n) return BINGO_E_CAPACITY;
    if (n) HIPCHK(hipEventSynchronize(g->ev[n]));
    for (uint32_t i = 0; i < n; ++i) HIPCHK(hipEventElapsedTime(&h_ms[i], g->ev[i], g->ev[i + 1]));
    return BINGO_OK;
}

void bingo_destroy(bingo_graph* g) {
    if (!g) return;
    release(g, hipDeviceSynchronize() == hipSuccess);
}

int bingo_trim(uint64_t* h_bytes) {
    const size_t given = dev_trim();
    if (h_bytes) *h_bytes = given;
    return BINGO_OK;
}

const char* bingo_strerror(int code) {
    switch (code) {
        case BINGO_OK: return "ok";
        case BINGO_E_INVALID: return "invalid argument";
        case BINGO_E_RANGE: return "vertex id out of range";
        case BINGO_E_WEIGHT: return "zero edge weight";
        case BINGO_E_OOM: return "device memory pool exhausted";
        case BINGO_E_CAPACITY: return "output buffer too small";
        case BINGO_E_HIP: return "HIP runtime error";
        case BINGO_E_INTERNAL: return "internal consistency check failed";
        default: return "unknown error";
    }
}

}  // extern "C"
