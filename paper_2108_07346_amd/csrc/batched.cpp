// Batched bridge queries: G independent graphs, one persistent launch.
//
// Host side of the batched path: plans the per-graph phase trees (chunks of
// chunk_edges edges, node regions, merge counters; for long lists a sample and
// runs), orders the work items largest-first, and captures "clear counters ->
// persistent kernel -> runs and finishes of the long lists" and "bridges of the
// graphs left over" in HIP graphs that are replayed while the batch shape and
// input buffer stay the same.  With the final step on the device the bridges come
// back; with final step 0 the certificates do, and a pool of host threads searches
// them.  Graphs past the small kernel's V go through plain queries over unions of
// them, those past a CU's LDS through one plain query each.  chunk_edges = 0 asks
// the library's tuner, which times candidate chunk sizes and workgroups per CU on
// the batch itself and remembers the winner per device and batch shape
// (tuner.cpp).
#include <algorithm>
#include <atomic>
#include <chrono>
#include <condition_variable>
#include <cstring>
#include <functional>
#include <map>
#include <memory>
#include <mutex>
#include <thread>

#include "internal.hpp"

namespace br {

namespace {

struct BatchPlan {
    // key
    int32_t G = 0, C = 0, bpc = 0;
    bool big = false;                // the class of graphs above the small kernel's V (160 KB kernel)
    std::vector<int64_t> eoff;
    std::vector<int32_t> V;
    // small graphs are the ones certified in LDS; the others go through br_bridges_find
    std::vector<int32_t> small, large;
    std::vector<int32_t> Mg;
    std::vector<int64_t> rbase, cbase, noff, ncap, items;
    std::vector<int32_t> stride, longs;
    std::vector<int64_t> sbase, fitems;
    int64_t nodes = 0, counters = 0, area0 = 0, cert_pairs = 0;
    // device memory: [clear block: ncnt | arrive | queue | err][meta][cert]
    void* dmem = nullptr;
    size_t clear_words = 0;
    BatchDev dev{};
    // pinned host: node-0 regions + node-0 counters + err
    void* hmem = nullptr;
    int2* h_area0 = nullptr;
    uint32_t* h_cnt0 = nullptr;
    uint32_t* h_err = nullptr;
    // first vertex of each small graph where their vertices are counted through
    // (roots' flags, the long graphs' states)
    std::vector<int64_t> vbase;      // [S+1]
    int64_t vtot = 0;
    // final step on the device: per graph bridge keys (u << 16 | v, sorted) in
    // one array; header word 0 = number of keys, words 16 + 2s, 17 + 2s = base
    // and count of small graph s; the keys follow the header directly
    uint32_t* d_sb = nullptr;
    uint32_t* h_sb = nullptr;
    int32_t* d_lists = nullptr;      // graphs left to the second kernel, by size class: [S] and [S]
    int32_t na = 0, nb = 0;
    int cus = 1;
    int64_t sb_hdr = 0;              // header words (16 + 2S)
    int64_t sb_keys = 0;             // room for keys: sum of (V_s - 1)
    size_t keys_hint = 0;            // keys of the previous call (size of the first copy)
    // captured launches: the persistent kernel, then (final step on the device)
    // the combined certificate and its bridge step, with an event in between
    hipGraph_t graph = nullptr, graph2 = nullptr;
    hipGraphExec_t exec = nullptr, exec2 = nullptr;
    const void* graph_edges = nullptr;
    int graph_mode = -1;
    int blocks = 0;
    bool owns = true;                // dmem / hmem allocated for this plan (else borrowed arenas)
    size_t dbytes = 0;
    ~BatchPlan() {
        if (exec) (void)hipGraphExecDestroy(exec);
        if (graph) (void)hipGraphDestroy(graph);
        if (exec2) (void)hipGraphExecDestroy(exec2);
        if (graph2) (void)hipGraphDestroy(graph2);
        if (owns && dmem) (void)hipFree(dmem);
        if (owns && hmem) (void)hipHostFree(hmem);
    }
};

struct BatchState {
    std::unique_ptr<Pool> pool;
    hipStream_t stream = nullptr;
    hipStream_t stream2 = nullptr;           // second branch of the captured final step (default priority)
    hipEvent_t fork = nullptr, join = nullptr;
    hipEvent_t ready = nullptr;              // the caller's stream has produced the input
    std::vector<std::unique_ptr<BatchPlan>> plans;      // small LRU
    std::vector<DfsScratch> scratch;
    std::vector<std::vector<uint64_t>> keys;
    std::unique_ptr<uint64_t[]> outk;           // per-graph bridge slots (reused, never zero-filled)
    size_t outk_n = 0;
    hipEvent_t e0 = nullptr, e1 = nullptr;
    hipEvent_t k0 = nullptr, k1 = nullptr;   // around the persistent kernel's graph (counter clear + kernel)
    hipEvent_t k2 = nullptr;                 // after the bridge step's graph
    // arenas of the plans built for one call only (serving), one per size
    // class: grown, never shrunk
    struct Arena {
        void* arena_d = nullptr;
        size_t arena_d_cap = 0;
        void* arena_h = nullptr;
        size_t arena_h_cap = 0;
    } arenas[2];
    std::unique_ptr<BatchPlan> transient[2];
    // graphs past the small kernel's V as disjoint unions: the edges of one and the
    // table that describes it (device, pinned host); at most kUnionEdges edges
    void *union_d = nullptr, *union_h = nullptr;
    size_t union_d_cap = 0, union_h_cap = 0;
};

BatchState* state_of(br_ctx* c) {
    if (!c->batched) c->batched = new BatchState();
    return static_cast<BatchState*>(c->batched);
}

int64_t part_lo(int64_t E, int64_t M, int64_t i) { return i * (E / M) + (i * (E % M)) / M; }

size_t a256(size_t x) { return (x + 255) & ~size_t(255); }

int64_t chunks_of(int64_t E, int32_t C) { return std::max<int64_t>(1, (E + C - 1) / C); }

// the same limit for every graph of up to batched_max_v_big() vertices, also those
// that are not split into chunks after all
int check_chunks(int32_t g, int64_t E, int32_t C) {
    const int64_t M = chunks_of(E, C);
    return M < (1 << 20) ? BR_OK : fail(BR_EINVAL, "batched: graph %d needs %lld chunks", g, (long long)M);
}

// Plan of one class of the batch: the small class takes the graphs with
// V <= batched_max_v_dev() (and lists those above batched_max_v_big() as
// `large`, for the plain path); the big class the graphs in between.
int build_plan(BatchPlan& P, const int64_t* eoff, const int32_t* V, int32_t G, int32_t C, int32_t bpc, int cus,
               bool big, BatchState::Arena* arena, hipStream_t upload) {
    P.G = G;
    P.C = C;
    P.bpc = bpc;
    P.big = big;
    P.eoff.assign(eoff, eoff + G + 1);
    P.V.assign(V, V + G);
    const int32_t lo = big ? batched_max_v_dev() : 0, hi = big ? batched_max_v_big() : batched_max_v_dev();
    for (int32_t g = 0; g < G; g++) {
        if (V[g] > lo && V[g] <= hi) P.small.push_back(g);
        else if (!big && V[g] > batched_max_v_big()) P.large.push_back(g);
    }
    const int32_t S = (int32_t)P.small.size();
    // per small graph (indexed by position s in P.small): chunks, nodes, counters
    P.Mg.resize(S);
    P.rbase.resize(S);
    P.cbase.resize(S);
    int64_t rest = S, ctr = 0;
    P.stride.assign(S, 0);
    P.sbase.assign((size_t)S + 1, 0);
    for (int32_t s = 0; s < S; s++) {
        const int64_t E = eoff[P.small[s] + 1] - eoff[P.small[s]], Vs = V[P.small[s]];
        // more than an item's edges, and at least twice the sample.  512 graphs
        // of 4,096 vertices in chunks of 32,768: 233 against 437 us in chunks
        // and merges at E = 9V, 304 against 829 at 32V (lists sorted by vertex
        // 313 against 500 and 338 against 871); 64 graphs 198 against 238 at 9V.
        // The sample: of E random edges 2(1 + d)exp(-d) have an end of degree
        // < 2 after dV/2 of them: 0.6% at 4V, less than V edges up to E = 128V;
        // past that 6V (0.02%)
        const bool is_long = !big && E > C && E >= 8 * Vs && E >= 2048;
        int64_t runs = 0;
        if (is_long) {
            const int64_t take = std::max<int64_t>((E >= 128 * Vs ? 6 : 4) * Vs, 1024);
            P.stride[s] = (int32_t)std::min<int64_t>(std::max<int64_t>(2, E / take), 1 << 30);
            P.longs.push_back(s);
            runs = (E + kLongRun - 1) / kLongRun;
            for (int64_t r = 0; r < runs; r++) P.fitems.push_back((int64_t)s << 32 | r);
        }
        // a run keeps at most what both forests take
        P.sbase[s + 1] = P.sbase[s] + std::min(E, 2 * runs * Vs);
        if (int rc = check_chunks(P.small[s], E, C)) return rc;
        const int64_t M = is_long ? 1 : chunks_of(E, C);
        P.Mg[s] = (int32_t)M;
        P.rbase[s] = rest;
        rest += M - 1;
        int R = 0;
        while ((int64_t(1) << R) < M) R++;
        P.cbase[s] = ctr;
        ctr += (int64_t)R * ((M + 1) / 2);
    }
    P.nodes = rest;
    P.counters = ctr;
    P.noff.assign(P.nodes, 0);
    P.ncap.assign(P.nodes, 0);
    // node-0 regions first (one contiguous copy to the host), then the others
    int64_t acc = 0;
    for (int pass = 0; pass < 2; pass++) {
        for (int32_t s = 0; s < S; s++) {
            const int32_t g = P.small[s];
            const int64_t E = eoff[g + 1] - eoff[g], M = P.Mg[s], bound = 2 * (int64_t(V[g]) - 1);
            for (int64_t i = (pass == 0 ? 0 : 1); i < (pass == 0 ? 1 : M); i++) {
                int64_t span = M;
                if (i) span = std::min<int64_t>(int64_t(1) << __builtin_ctzll((unsigned long long)i), M - i);
                const int64_t cap = std::min(part_lo(E, M, std::min<int64_t>(M, i + span)) - part_lo(E, M, i), bound);
                const int64_t idx = i ? P.rbase[s] + i - 1 : s;
                P.noff[idx] = acc;
                P.ncap[idx] = cap;
                acc += cap;
            }
        }
        if (pass == 0) P.area0 = acc;
    }
    P.cert_pairs = acc;
    // items, largest chunk first (ties: graph order)
    struct It { int64_t len, code; };
    std::vector<It> its;
    for (int32_t s = 0; s < S; s++) {
        const int32_t g = P.small[s];
        const int64_t E = eoff[g + 1] - eoff[g], M = P.Mg[s];
        for (int64_t k = 0; k < M; k++)
            its.push_back({(part_lo(E, M, k + 1) - part_lo(E, M, k)) / std::max(P.stride[s], 1), ((int64_t)s << 20) | k});
    }
    std::stable_sort(its.begin(), its.end(), [](const It& a, const It& b) { return a.len > b.len; });
    P.items.resize(its.size());
    for (size_t i = 0; i < its.size(); i++) P.items[i] = its[i].code;
    // device memory: [clear block | metadata uploaded in one copy | the rest]
    P.clear_words = 2 * (size_t)P.nodes + (size_t)P.counters + 2 + (size_t)S;
    P.vbase.assign((size_t)S + 1, 0);
    for (int32_t s = 0; s < S; s++) P.vbase[s + 1] = P.vbase[s] + V[P.small[s]];
    P.vtot = P.vbase[S];
    if (P.vtot >= (int64_t(1) << 30)) return fail(BR_EINVAL, "batched: %lld vertices in one batch", (long long)P.vtot);
    P.sb_hdr = 16 + 2 * (int64_t)S;
    P.sb_keys = std::max<int64_t>(1, P.vtot - S);   // sum of (V_s - 1): every bridge of every graph
    const size_t o_clear = 0;
    size_t o = a256(o_clear + 4 * P.clear_words);
    const size_t o_meta = o;
    const size_t o_eoff = o; o = a256(o + 8 * 2 * (size_t)std::max(S, 1));
    const size_t o_V = o; o = a256(o + 4 * (size_t)S);
    const size_t o_M = o; o = a256(o + 4 * (size_t)S);
    const size_t o_rb = o; o = a256(o + 8 * (size_t)S);
    const size_t o_cb = o; o = a256(o + 8 * (size_t)S);
    const size_t o_noff = o; o = a256(o + 8 * (size_t)P.nodes);
    const size_t o_ncap = o; o = a256(o + 8 * (size_t)P.nodes);
    const size_t o_items = o; o = a256(o + 8 * std::max<size_t>(P.items.size(), 1));
    const size_t o_vb = o; o = a256(o + 8 * (size_t)(S + 1));
    const size_t o_stride = o; o = a256(o + 4 * (size_t)std::max(S, 1));
    const size_t o_sbase = o; o = a256(o + 8 * (size_t)(S + 1));
    const size_t o_fitems = o; o = a256(o + 8 * std::max<size_t>(P.fitems.size(), 1));
    const size_t o_longs = o; o = a256(o + 4 * std::max<size_t>(P.longs.size(), 1));
    const size_t meta_bytes = o - o_meta;
    const size_t o_lists = o; if (!big) o = a256(o + 8 * (size_t)std::max(S, 1));
    const size_t o_cert = o; o = a256(o + 8 * (size_t)std::max<int64_t>(P.cert_pairs, 1));
    const size_t o_root = o; o = a256(o + 4 * (size_t)std::max<int64_t>(P.vtot, 1));
    const bool any_long = !P.longs.empty();
    const size_t o_stq = o; if (any_long) o = a256(o + 4 * (size_t)P.vtot);
    const size_t o_surv = o; if (any_long) o = a256(o + 4 * (size_t)P.sbase[S]);
    const size_t o_sb = o; if (!big) o = a256(o + 4 * (size_t)(P.sb_hdr + P.sb_keys));
    // pinned host staging: node-0 regions, node-0 counters, error word, keys;
    // then room for the metadata's one upload
    const size_t h_keys = a256(8 * (size_t)std::max<int64_t>(P.area0, 1)) + a256(8 * (size_t)std::max(S, 1)) + 256;
    const size_t h_meta = h_keys + (big ? 0 : a256(4 * (size_t)(P.sb_hdr + P.sb_keys)));
    const size_t hbytes = h_meta + a256(meta_bytes);
    if (arena) {
        // a plan for one call: the batch state's arenas (grown when too small)
        if (arena->arena_d_cap < o) {
            if (arena->arena_d) BR_HIP(hipFree(arena->arena_d));
            arena->arena_d = nullptr;
            arena->arena_d_cap = 0;
            BR_HIP(hipMalloc(&arena->arena_d, o));
            arena->arena_d_cap = o;
        }
        if (arena->arena_h_cap < hbytes) {
            if (arena->arena_h) BR_HIP(hipHostFree(arena->arena_h));
            arena->arena_h = nullptr;
            arena->arena_h_cap = 0;
            BR_HIP(hipHostMalloc(&arena->arena_h, hbytes, hipHostMallocDefault));
            arena->arena_h_cap = hbytes;
        }
        P.dmem = arena->arena_d;
        P.hmem = arena->arena_h;
        P.owns = false;
    } else {
        BR_HIP(hipMalloc(&P.dmem, o));
        BR_HIP(hipHostMalloc(&P.hmem, hbytes, hipHostMallocDefault));
        P.owns = true;
    }
    P.dbytes = o;
    char* d = static_cast<char*>(P.dmem);
    char* h = static_cast<char*>(P.hmem);
    {
        // metadata assembled in pinned memory with the device layout, one copy
        char* m = h + h_meta;
        auto put = [&](size_t off, const void* src, size_t n) { if (n) std::memcpy(m + (off - o_meta), src, n); };
        std::vector<int32_t> sV(S);
        std::vector<int64_t> se2(2 * (size_t)S);     // graph s: edges [se2[2s], se2[2s+1])
        for (int32_t s = 0; s < S; s++) {
            sV[s] = V[P.small[s]];
            se2[2 * s] = eoff[P.small[s]];
            se2[2 * s + 1] = eoff[P.small[s] + 1];
        }
        put(o_eoff, se2.data(), 8 * 2 * (size_t)S);
        put(o_V, sV.data(), 4 * (size_t)S);
        put(o_M, P.Mg.data(), 4 * (size_t)S);
        put(o_rb, P.rbase.data(), 8 * (size_t)S);
        put(o_cb, P.cbase.data(), 8 * (size_t)S);
        put(o_noff, P.noff.data(), 8 * (size_t)P.nodes);
        put(o_ncap, P.ncap.data(), 8 * (size_t)P.nodes);
        put(o_items, P.items.data(), 8 * P.items.size());
        put(o_vb, P.vbase.data(), 8 * (size_t)S);
        put(o_stride, P.stride.data(), 4 * (size_t)S);
        put(o_sbase, P.sbase.data(), 8 * (size_t)(S + 1));
        put(o_fitems, P.fitems.data(), 8 * P.fitems.size());
        put(o_longs, P.longs.data(), 4 * P.longs.size());
        if (!big)
            for (int32_t s = 0; s < S; s++) (V[P.small[s]] <= small_bridges_split_v() ? P.na : P.nb)++;
        // ordered before the plan's launches (the same stream); the pinned
        // source is rewritten only by a later call, after that call's wait
        BR_HIP(hipMemcpyAsync(d + o_meta, m, meta_bytes, hipMemcpyHostToDevice, upload));
    }
    P.d_sb = reinterpret_cast<uint32_t*>(d + o_sb);
    P.d_lists = reinterpret_cast<int32_t*>(d + o_lists);
    P.cus = std::max(1, cus);
    uint32_t* clr = reinterpret_cast<uint32_t*>(d + o_clear);
    P.dev.eoff = reinterpret_cast<const int64_t*>(d + o_eoff);
    P.dev.V = reinterpret_cast<const int32_t*>(d + o_V);
    P.dev.Mg = reinterpret_cast<const int32_t*>(d + o_M);
    P.dev.rbase = reinterpret_cast<const int64_t*>(d + o_rb);
    P.dev.cbase = reinterpret_cast<const int64_t*>(d + o_cb);
    P.dev.noff = reinterpret_cast<const int64_t*>(d + o_noff);
    P.dev.ncap = reinterpret_cast<const int64_t*>(d + o_ncap);
    P.dev.items = reinterpret_cast<const int64_t*>(d + o_items);
    P.dev.n_items = (int64_t)P.items.size();
    P.dev.cert = reinterpret_cast<int2*>(d + o_cert);
    P.dev.ncnt = clr;
    P.dev.arrive = clr + 2 * P.nodes;
    P.dev.queue = clr + 2 * P.nodes + P.counters;
    P.dev.err = P.dev.queue + 1;
    P.dev.scnt = P.dev.err + 1;
    P.dev.stride = any_long ? reinterpret_cast<const int32_t*>(d + o_stride) : nullptr;
    P.dev.sbase = reinterpret_cast<const int64_t*>(d + o_sbase);
    P.dev.fitems = reinterpret_cast<const int64_t*>(d + o_fitems);
    P.dev.longs = reinterpret_cast<const int32_t*>(d + o_longs);
    P.dev.stq = reinterpret_cast<uint32_t*>(d + o_stq);
    P.dev.surv = reinterpret_cast<uint32_t*>(d + o_surv);
    P.dev.n_fitems = (int64_t)P.fitems.size();
    P.dev.n_long = (int32_t)P.longs.size();
    P.dev.vbase = reinterpret_cast<const int64_t*>(d + o_vb);
    P.dev.rootw = reinterpret_cast<uint32_t*>(d + o_root);
    P.h_area0 = reinterpret_cast<int2*>(h);
    P.h_cnt0 = reinterpret_cast<uint32_t*>(h + a256(8 * (size_t)std::max<int64_t>(P.area0, 1)));
    P.h_err = P.h_cnt0 + 2 * (size_t)std::max(S, 1);
    P.h_sb = reinterpret_cast<uint32_t*>(h + a256(8 * (size_t)std::max<int64_t>(P.area0, 1)) +
                                         a256(8 * (size_t)std::max(S, 1)) + 256);
    // the big class fills one workgroup per CU (its LDS)
    P.blocks = std::max(1, big ? cus : cus * bpc);
    return BR_OK;
}

// The captured parts.  0: clear the counters, the persistent kernel, the long
// lists' runs and finishes.  1 (final step on the device): the bridges of the graphs
// that the kernel left, by size class.
int enqueue(BatchPlan& P, const int32_t* d_edges, hipStream_t s, int mode, int part, BatchState* st) {
    P.dev.edges = reinterpret_cast<const int2*>(d_edges);
    if (part == 0) {
        launch_fill_u32(P.dev.ncnt, (int64_t)P.clear_words, 0u, s);
        const bool fin = mode == 1 && !P.big;
        P.dev.out_hdr = fin ? P.d_sb : nullptr;
        P.dev.out_keys = P.d_sb + P.sb_hdr;
        P.dev.list_a = P.d_lists;
        P.dev.list_b = P.d_lists + P.small.size();
        P.dev.split_v = small_bridges_split_v();
        if (fin) launch_fill_u32(P.d_sb, 16, 0u, s);
        BR_HIP(hipGetLastError());
        if (P.dev.n_items) launch_batched(P.dev, P.blocks, s, P.big);
        launch_batched_long(P.dev, s);
        BR_HIP(hipGetLastError());
        return BR_OK;
    }
    if (mode == 1 && !P.small.empty()) {
        // fork: the two size classes run side by side, then join back on s
        BR_HIP(hipEventRecord(st->fork, s));
        BR_HIP(hipStreamWaitEvent(st->stream2, st->fork, 0));
        launch_small_bridges(P.dev, P.na, P.nb, P.cus, s, st->stream2);
        BR_HIP(hipGetLastError());
        BR_HIP(hipEventRecord(st->join, st->stream2));
        BR_HIP(hipStreamWaitEvent(s, st->join, 0));
    }
    return BR_OK;
}

// node-0 certificates (or, with the final step on the device, the number of
// bridges), their counters and the error word to the host
int copy_back(BatchPlan& P, hipStream_t s, int mode) {
    const int32_t S = (int32_t)P.small.size();
    if (mode == 1) {
        if (S) {
            // header, per-graph table and the first keys in one copy
            const size_t guess = std::min<size_t>(std::max<size_t>(P.keys_hint, 4096), (size_t)P.sb_keys);
            BR_HIP(hipMemcpyAsync(P.h_sb, P.d_sb, 4 * ((size_t)P.sb_hdr + guess), hipMemcpyDeviceToHost, s));
        }
        BR_HIP(hipMemcpyAsync(P.h_err, P.dev.err, 4, hipMemcpyDeviceToHost, s));
        return BR_OK;
    }
    if (P.area0) BR_HIP(hipMemcpyAsync(P.h_area0, P.dev.cert, 8 * (size_t)P.area0, hipMemcpyDeviceToHost, s));
    if (S) BR_HIP(hipMemcpyAsync(P.h_cnt0, P.dev.ncnt, 8 * (size_t)S, hipMemcpyDeviceToHost, s));
    BR_HIP(hipMemcpyAsync(P.h_err, P.dev.err, 4, hipMemcpyDeviceToHost, s));
    return BR_OK;
}

static int capture(BatchPlan& P, const int32_t* d_edges, hipStream_t s, int mode, int part, hipGraph_t* graph,
                   hipGraphExec_t* exec, BatchState* st) {
    BR_HIP(hipStreamBeginCapture(s, hipStreamCaptureModeThreadLocal));
    int rc = enqueue(P, d_edges, s, mode, part, st);
    hipGraph_t g = nullptr;
    const hipError_t e = hipStreamEndCapture(s, &g);
    if (rc) {
        if (g) (void)hipGraphDestroy(g);
        return rc;
    }
    if (e != hipSuccess) return hip_fail(e, "hipStreamEndCapture");
    *graph = g;
    BR_HIP(hipGraphInstantiate(exec, g, nullptr, nullptr, 0));
    return BR_OK;
}

int run_device(BatchState& st, BatchPlan& P, const int32_t* d_edges, int mode, bool captured = true) {
    hipStream_t s = st.stream;
    const bool two = mode == 1 && !P.small.empty();
    if (!captured) {
        // a plan used once: the launches go straight to the stream
        BR_HIP(hipEventRecord(st.k0, s));
        int rc = enqueue(P, d_edges, s, mode, 0, &st);
        if (rc) return rc;
        BR_HIP(hipEventRecord(st.k1, s));
        if (two) {
            rc = enqueue(P, d_edges, s, mode, 1, &st);
            if (rc) return rc;
        }
        BR_HIP(hipEventRecord(st.k2, s));
        return copy_back(P, s, mode);
    }
    if (!(P.exec && P.graph_edges == d_edges && P.graph_mode == mode)) {
        for (hipGraphExec_t* x : {&P.exec, &P.exec2})
            if (*x) { (void)hipGraphExecDestroy(*x); *x = nullptr; }
        for (hipGraph_t* g : {&P.graph, &P.graph2})
            if (*g) { (void)hipGraphDestroy(*g); *g = nullptr; }
        P.graph_edges = nullptr;
        int rc = capture(P, d_edges, s, mode, 0, &P.graph, &P.exec, &st);
        if (rc) return rc;
        if (two) {
            rc = capture(P, d_edges, s, mode, 1, &P.graph2, &P.exec2, &st);
            if (rc) return rc;
        }
        P.graph_edges = d_edges;
        P.graph_mode = mode;
    }
    BR_HIP(hipEventRecord(st.k0, s));
    BR_HIP(hipGraphLaunch(P.exec, s));
    BR_HIP(hipEventRecord(st.k1, s));
    if (two) BR_HIP(hipGraphLaunch(P.exec2, s));
    BR_HIP(hipEventRecord(st.k2, s));
    return copy_back(P, s, mode);
}

std::string shape_key(int device, const int64_t* eoff, const int32_t* V, int32_t G) {
    // batch shape bucket for the tuner: device arch, G, total edges and
    // largest V (log2 buckets)
    int64_t E = eoff[G] - eoff[0];
    int32_t mv = 0;
    for (int32_t g = 0; g < G; g++) mv = std::max(mv, V[g]);
    return arch_name(device) + "|batched|g" + std::to_string(log2_bucket(G)) + "|e" + std::to_string(log2_bucket(E)) +
           "|v" + std::to_string(log2_bucket(mv)) + kTuneGen;
}

bool same_shape(const BatchPlan& P, const int64_t* eoff, const int32_t* V, int32_t G, int32_t C, int32_t bpc, bool big) {
    return P.G == G && P.C == C && P.bpc == bpc && P.big == big && std::equal(P.eoff.begin(), P.eoff.end(), eoff) &&
           std::equal(P.V.begin(), P.V.end(), V);
}

}  // namespace

size_t batched_device_bytes(br_ctx* c) {
    if (!c->batched) return 0;
    auto* st = static_cast<BatchState*>(c->batched);
    size_t n = 0;
    for (auto& a : st->arenas) n += a.arena_d_cap;
    for (auto& P : st->plans)
        if (P->owns) n += P->dbytes;
    return n + st->union_d_cap;
}

void batched_release(br_ctx* c) {
    if (!c->batched) return;
    auto* st = static_cast<BatchState*>(c->batched);
    if (st->stream) (void)hipStreamSynchronize(st->stream);
    st->plans.clear();
    for (auto& t : st->transient) t.reset();
    for (auto& a : st->arenas) {
        if (a.arena_d) (void)hipFree(a.arena_d);
        if (a.arena_h) (void)hipHostFree(a.arena_h);
    }
    if (st->union_d) (void)hipFree(st->union_d);
    if (st->union_h) (void)hipHostFree(st->union_h);
    if (st->e0) (void)hipEventDestroy(st->e0);
    if (st->e1) (void)hipEventDestroy(st->e1);
    if (st->k0) (void)hipEventDestroy(st->k0);
    if (st->k1) (void)hipEventDestroy(st->k1);
    if (st->k2) (void)hipEventDestroy(st->k2);
    if (st->fork) (void)hipEventDestroy(st->fork);
    if (st->join) (void)hipEventDestroy(st->join);
    if (st->ready) (void)hipEventDestroy(st->ready);
    if (st->stream2) (void)hipStreamDestroy(st->stream2);
    if (st->stream) (void)hipStreamDestroy(st->stream);
    delete st;
    c->batched = nullptr;
}

// Bridges of every graph of a big-class plan after its launches completed, by
// Algorithm 1 per graph on the host; out[k] = pairs of graph small[k].
static int gather_big(BatchState& st, BatchPlan& P, std::vector<std::vector<int32_t>>& out) {
    const int32_t S = (int32_t)P.small.size();
    out.assign(S, {});
    std::atomic<int32_t> next{0};
    std::atomic<int> bad{0};
    st.pool->run([&](int w) {
        DfsScratch& sc = st.scratch[w];
        std::vector<uint64_t>& keys = st.keys[w];
        for (;;) {
            const int32_t s = next.fetch_add(1);
            if (s >= S) break;
            const uint32_t n1 = P.h_cnt0[2 * s], n2 = P.h_cnt0[2 * s + 1];
            const int64_t off = P.noff[s], capg = P.ncap[s];
            if ((int64_t)n1 + n2 > capg) {
                bad = 1;
                continue;
            }
            keys.clear();
            certificate_bridges(P.h_area0 + off, n1, P.h_area0 + off + capg - n2, n2, P.V[P.small[s]], sc, keys);
            canonical_sort(keys);
            for (uint64_t k : keys) {
                out[s].push_back((int32_t)(k >> 32));
                out[s].push_back((int32_t)(k & 0xffffffffu));
            }
        }
    });
    if (bad) return fail(BR_EINTERNAL, "batched: certificate counts exceed their region");
    return BR_OK;
}

// Bridges of the graphs gs (indices into the batch) through plain queries over
// disjoint unions of them; out[k] = pairs of graph gs[k].  Per graph the 160 KB
// kernel took a CU for its chunks and merges in turn (150 graphs of 100 to
// 24,000 vertices: 1,040 of 1,860 us); the union gives every CU edges of all
// of them.  A union is a copy of its graphs' edges, so it is kept to 1 GiB (the query
// over one takes 0.3 ms and more whatever its size, the copy 0.4); a graph that
// stands alone, as one past that does, is queried where it lies.
constexpr int64_t kUnionRun = 64;        // rows per workgroup of the list's long part (32,768 edges per table)
constexpr int64_t kUnionEdges = int64_t(1) << 27;
static int find_union(br_ctx* c, BatchState& st, const int32_t* d_edges, const int64_t* eoff, const int32_t* V,
                      const std::vector<int32_t>& gs, std::vector<std::vector<int32_t>>& out) {
    const int32_t n = (int32_t)gs.size();
    out.assign(n, {});
    for (int32_t k0 = 0; k0 < n;) {
        // as many graphs as the final step takes vertices
        int64_t vt = 0, et = 0, longest = 0;
        int32_t k1 = k0;
        std::vector<int64_t> vbase, at;
        std::vector<RowItem> rows;       // runs of rows of one graph: a workgroup's share of the list
        int32_t max_v = 0;
        const int64_t row = kRow;
        while (k1 < n && vt + V[gs[k1]] <= kFinalStepMaxV) {
            const int64_t m = eoff[gs[k1] + 1] - eoff[gs[k1]], nr = (m + row - 1) / row;
            if (k1 > k0 && et + nr * row > kUnionEdges) break;
            vbase.push_back(vt);
            at.push_back(et);
            for (int64_t r = 0; r < nr; r += kUnionRun)
                rows.push_back(RowItem{(uint32_t)(et / row + r), (uint32_t)(et / row + std::min(nr, r + kUnionRun)), (int32_t)vt,
                                       V[gs[k1]]});
            vt += V[gs[k1]];
            et += nr * row;
            max_v = std::max(max_v, V[gs[k1]]);
            longest = std::max(longest, m);
            k1++;
        }
        vbase.push_back(vt);
        (k1 - k0 == 1 ? c->route.alone : c->route.in_unions) += k1 - k0;
        if (k1 - k0 == 1) {
            const int32_t g = gs[k0];
            const TuneEntry knobs{{"fuse", 1}};
            out[k0].resize(2 * (size_t)(V[g] - 1));
            int64_t nb = 0;
            const int rc = bridges_find(c, d_edges + 2 * eoff[g], eoff[g + 1] - eoff[g], V[g], 1, out[k0].data(), V[g] - 1, &nb,
                                        st.stream, &knobs);
            if (rc == BR_ERANGE) return fail(BR_ERANGE, "batched: an edge has a vertex id outside its graph's [0, V)");
            if (rc) return rc;
            out[k0].resize(2 * (size_t)nb);
            k0 = k1;
            continue;
        }
        const size_t ebytes = a256(8 * (size_t)et), rbytes = a256(sizeof(RowItem) * rows.size());
        const size_t tbytes = rbytes + sizeof(UnionItem) * (size_t)(k1 - k0);
        if (st.union_d_cap < ebytes + tbytes) {
            BR_HIP(hipStreamSynchronize(st.stream));
            if (st.union_d) BR_HIP(hipFree(st.union_d));
            st.union_d = nullptr;
            st.union_d_cap = 0;
            BR_HIP(hipMalloc(&st.union_d, ebytes + tbytes));
            st.union_d_cap = ebytes + tbytes;
        }
        if (st.union_h_cap < tbytes) {
            if (st.union_h) BR_HIP(hipHostFree(st.union_h));
            st.union_h = nullptr;
            st.union_h_cap = 0;
            BR_HIP(hipHostMalloc(&st.union_h, tbytes, hipHostMallocDefault));
            st.union_h_cap = tbytes;
        }
        std::copy(rows.begin(), rows.end(), static_cast<RowItem*>(st.union_h));
        UnionItem* it = reinterpret_cast<UnionItem*>(static_cast<char*>(st.union_h) + rbytes);
        for (int32_t k = k0; k < k1; k++) {
            const int32_t g = gs[k];
            it[k - k0] = UnionItem{d_edges + 2 * eoff[g], at[k - k0], eoff[g + 1] - eoff[g], (int32_t)vbase[k - k0], V[g]};
        }
        int32_t* du = static_cast<int32_t*>(st.union_d);
        char* dt = static_cast<char*>(st.union_d) + ebytes;
        BR_HIP(hipMemcpyAsync(dt, st.union_h, tbytes, hipMemcpyHostToDevice, st.stream));
        launch_union_edges(reinterpret_cast<const UnionItem*>(dt + rbytes), k1 - k0, longest, (int32_t)row, du, st.stream);
        BR_HIP(hipGetLastError());
        c->fused.items = reinterpret_cast<const RowItem*>(dt);
        c->fused.n_items = (int32_t)rows.size();
        c->fused.item_words = (int32_t)(((max_v + 1) / 2 + 3) & ~3);
        const TuneEntry knobs{{"fuse", 1}, {"table", 0}};
        std::vector<int32_t> pairs(2 * (size_t)std::max<int64_t>(vt - (k1 - k0), 1));
        int64_t nb = 0;
        const int rc = bridges_find(c, du, et, (int32_t)vt, 1, pairs.data(), (int64_t)pairs.size() / 2, &nb, st.stream, &knobs);
        c->fused.items = nullptr;          // this union's rows: no other call may take them
        c->fused.n_items = 0;
        if (rc == BR_ERANGE) return fail(BR_ERANGE, "batched: an edge has a vertex id outside its graph's [0, V)");
        if (rc) return rc;
        // ascending: each graph's pairs are one run
        int32_t k = k0;
        for (int64_t i = 0; i < nb; i++) {
            const int64_t u = pairs[2 * i], v = pairs[2 * i + 1];
            while (k + 1 < k1 && vbase[k + 1 - k0] <= u) k++;
            const int64_t b = vbase[k - k0];
            if (u < b || v >= vbase[k + 1 - k0]) return fail(BR_EINTERNAL, "batched: a bridge joins two graphs");
            out[k].push_back((int32_t)(u - b));
            out[k].push_back((int32_t)(v - b));
        }
        k0 = k1;
    }
    return BR_OK;
}

static int get_plan(br_ctx* c, BatchState& st, const int64_t* eoff, const int32_t* V, int32_t G, int32_t C,
                    int32_t bpc, BatchPlan** out, bool big = false) {
    for (size_t i = 0; i < st.plans.size(); i++) {
        if (same_shape(*st.plans[i], eoff, V, G, C, bpc, big)) {
            std::rotate(st.plans.begin(), st.plans.begin() + i, st.plans.begin() + i + 1);
            *out = st.plans[0].get();
            return BR_OK;
        }
    }
    hipDeviceProp_t prop;
    BR_HIP(hipGetDeviceProperties(&prop, c->device));
    auto P = std::make_unique<BatchPlan>();
    int rc = build_plan(*P, eoff, V, G, C, bpc, prop.multiProcessorCount, big, nullptr, st.stream);
    if (rc) return rc;
    st.plans.insert(st.plans.begin(), std::move(P));
    if (st.plans.size() > 4) st.plans.pop_back();
    *out = st.plans[0].get();
    return BR_OK;
}

// a plan for one call of a batch shape not worth keeping (serving): built in
// the class's arena, never captured
static int get_transient(br_ctx* c, BatchState& st, const int64_t* eoff, const int32_t* V, int32_t G, int32_t C,
                         int32_t bpc, BatchPlan** out, bool big) {
    const int k = big ? 1 : 0;
    st.transient[k].reset(new BatchPlan());
    const int cus = g_cus > 0 ? g_cus : 256;
    int rc = build_plan(*st.transient[k], eoff, V, G, C, bpc, cus, big, &st.arenas[k], st.stream);
    if (rc) return rc;
    *out = st.transient[k].get();
    return BR_OK;
}

int batched_query(br_ctx* c, const int32_t* d_edges, const int64_t* h_edge_off, const int32_t* h_V, int32_t G,
                  int32_t chunk_edges, int32_t* h_bridges, int64_t cap, int64_t* h_bridge_off, void* stream,
                  bool transient) {
    auto t0 = std::chrono::steady_clock::now();
    BR_HIP(hipSetDevice(c->device));
    BatchState& st = *state_of(c);
    if (!st.stream) {
        BR_HIP(hipStreamCreateWithFlags(&st.stream, hipStreamNonBlocking));
        BR_HIP(hipEventCreate(&st.e0));
        BR_HIP(hipEventCreate(&st.e1));
        BR_HIP(hipEventCreate(&st.k0));
        BR_HIP(hipEventCreate(&st.k1));
        BR_HIP(hipEventCreate(&st.k2));
        BR_HIP(hipStreamCreateWithFlags(&st.stream2, hipStreamNonBlocking));
        BR_HIP(hipEventCreateWithFlags(&st.fork, hipEventDisableTiming));
        BR_HIP(hipEventCreateWithFlags(&st.join, hipEventDisableTiming));
        BR_HIP(hipEventCreateWithFlags(&st.ready, hipEventDisableTiming));
        if (prepare_small_bridges() != 0) return fail(BR_EHIP, "batched: cannot raise the LDS limit of the bridge kernel");
        if (small_bridges_max_v() < batched_max_v_dev()) return fail(BR_EINTERNAL, "batched: bridge kernel limit below the LDS path's");
    }
    if (!st.pool) {
        int n = (int)std::thread::hardware_concurrency();
        n = std::max(1, std::min(n, 16));
        st.pool = std::make_unique<Pool>(n);
        st.scratch.resize(n);
        st.keys.resize(n);
    }
    // the caller's stream must have produced the input
    BR_HIP(hipEventRecord(st.ready, static_cast<hipStream_t>(stream)));
    BR_HIP(hipStreamWaitEvent(st.stream, st.ready, 0));

    // chunk size and workgroups per CU: given, or the tuner's (measured on
    // this batch the first time its shape bucket is seen on this device,
    // and kept in BR_AUTOTUNE_CACHE when that names a file)
    int32_t C = chunk_edges, bpc = batched_blocks_per_cu();
    if (C == 0) {
        const std::string key = shape_key(c->device, h_edge_off, h_V, G);
        TuneEntry t;
        if (tune_get(key, t) && t.count("chunk_edges") && t.count("blocks_per_cu")) {
            C = (int32_t)t["chunk_edges"];
            bpc = (int32_t)t["blocks_per_cu"];
        } else if (transient) {
            C = 32768;            // nothing measured for this shape yet: no time to measure now
        } else {
            // time every candidate on this batch (device part only)
            float best = 1e30f;
            int32_t bestC = 16384, bestB = bpc;
            for (int32_t b = 1; b <= batched_max_blocks_per_cu(); b++)
                for (int32_t cand : {4096, 8192, 16384, 32768, 65536, 131072}) {
                    BatchPlan* P = nullptr;
                    int rc = get_plan(c, st, h_edge_off, h_V, G, cand, b, &P);
                    if (rc) return rc;
                    float ms = 1e30f;
                    for (int rep = 0; rep < 3; rep++) {
                        BR_HIP(hipEventRecord(st.e0, st.stream));
                        rc = run_device(st, *P, d_edges, 0);
                        if (rc) return rc;
                        BR_HIP(hipEventRecord(st.e1, st.stream));
                        BR_HIP(hipEventSynchronize(st.e1));
                        float f = 0.f;
                        BR_HIP(hipEventElapsedTime(&f, st.e0, st.e1));
                        if (rep > 0) ms = std::min(ms, f);
                    }
                    if (ms < best) {
                        best = ms;
                        bestC = cand;
                        bestB = b;
                    }
                }
            tune_put(key, {{"chunk_edges", bestC}, {"blocks_per_cu", bestB}, {"ms", best}});
            C = bestC;
            bpc = bestB;
        }
    }
    BatchPlan* P = nullptr;
    int rc = transient ? get_transient(c, st, h_edge_off, h_V, G, C, bpc, &P, false)
                       : get_plan(c, st, h_edge_off, h_V, G, C, bpc, &P);
    if (rc) return rc;
    // graphs above the small kernel's V and within a CU's LDS: one query over
    // their union (final step on the device), or the 160 KB kernel, one
    // workgroup per CU, and the host's search of each certificate
    const int mode = c->final_step;
    BatchPlan* PM = nullptr;
    std::vector<int32_t> mid;
    for (int32_t g = 0; g < G; g++)
        if (h_V[g] > batched_max_v_dev() && h_V[g] <= batched_max_v_big()) {
            if ((rc = check_chunks(g, h_edge_off[g + 1] - h_edge_off[g], C))) return rc;
            mid.push_back(g);
        }
    if (!mid.empty() && mode != 1) {
        rc = transient ? get_transient(c, st, h_edge_off, h_V, G, C, 1, &PM, true)
                       : get_plan(c, st, h_edge_off, h_V, G, C, 1, &PM, true);
        if (rc) return rc;
    }
    if (c->profiling) BR_HIP(hipEventRecord(st.e0, st.stream));
    rc = run_device(st, *P, d_edges, mode, !transient);
    if (rc) return rc;
    if (PM) {
        rc = run_device(st, *PM, d_edges, mode, !transient);
        if (rc) return rc;
    }
    std::vector<std::vector<int32_t>> mid_out;
    c->route.longs = (int64_t)P->longs.size();
    c->route.in_unions = c->route.alone = 0;
    if (!mid.empty() && mode == 1) {
        rc = find_union(c, st, d_edges, h_edge_off, h_V, mid, mid_out);
        if (rc) {
            (void)hipStreamSynchronize(st.stream);
            return rc;
        }
    }
    if (c->profiling) BR_HIP(hipEventRecord(st.e1, st.stream));
    BR_HIP(hipStreamSynchronize(st.stream));
    auto t1 = std::chrono::steady_clock::now();
    for (BatchPlan* Q : {P, PM}) {
        if (!Q) continue;
        if (*Q->h_err & 1u) return fail(BR_ERANGE, "batched: an edge has a vertex id outside its graph's [0, V)");
        if (*Q->h_err) return fail(BR_EINTERNAL, "batched: certificate region overflow");
    }
    if (PM) {
        rc = gather_big(st, *PM, mid_out);
        if (rc) return rc;
    }

    // final search per small graph; bridges of graph g go to a slot of V_g - 1
    // pairs, compacted afterwards
    const int32_t S = (int32_t)P->small.size();
    std::vector<int64_t> slot(S + 1, 0), nb(G, 0);
    for (size_t k = 0; k < mid.size(); k++) nb[mid[k]] = (int64_t)mid_out[k].size() / 2;
    for (int32_t s = 0; s < S; s++) slot[s + 1] = slot[s] + std::max(P->V[P->small[s]] - 1, 0);
    uint64_t* outk = nullptr;
    const uint32_t* keys = nullptr;     // mode 1: the device's sorted keys, (u | v << 16)
    if (mode != 1) {
        if (st.outk_n < (size_t)std::max<int64_t>(slot[S], 1)) {
            st.outk_n = (size_t)std::max<int64_t>(slot[S], 1);
            st.outk.reset(new uint64_t[st.outk_n]);
        }
        outk = st.outk.get();
    }
    if (mode == 1) {
        // per graph: base and count in the key array, keys already sorted
        const size_t guess = std::min<size_t>(std::max<size_t>(P->keys_hint, 4096), (size_t)P->sb_keys);
        const uint32_t* hdr = P->h_sb;
        keys = P->h_sb + P->sb_hdr;
        const uint32_t nk = S ? hdr[0] : 0;
        if (nk > (uint32_t)P->sb_keys) return fail(BR_EINTERNAL, "batched: %u bridge keys for room %lld", nk, (long long)P->sb_keys);
        if (nk > guess) {
            BR_HIP(hipMemcpyAsync(P->h_sb + P->sb_hdr + guess, P->d_sb + P->sb_hdr + guess, 4 * (size_t)(nk - guess),
                                  hipMemcpyDeviceToHost, st.stream));
            BR_HIP(hipStreamSynchronize(st.stream));
        }
        P->keys_hint = nk;
        // counts only here; the keys go straight to the caller's array below
        for (int32_t s = 0; s < S; s++) {
            const uint32_t base = hdr[16 + 2 * s], cnt = hdr[17 + 2 * s];
            if ((uint64_t)base + cnt > nk || (int64_t)cnt > slot[s + 1] - slot[s])
                return fail(BR_EINTERNAL, "batched: graph %d reports %u bridges at %u", (int)P->small[s], cnt, base);
            nb[P->small[s]] = cnt;
        }
    } else {
        std::atomic<int32_t> next{0};
        std::atomic<int> bad{0};
        st.pool->run([&](int w) {
            DfsScratch& sc = st.scratch[w];
            std::vector<uint64_t>& keys = st.keys[w];
            for (;;) {
                const int32_t s = next.fetch_add(1);
                if (s >= S) break;
                const int32_t g = P->small[s];
                const uint32_t n1 = P->h_cnt0[2 * s], n2 = P->h_cnt0[2 * s + 1];
                const int64_t off = P->noff[s], capg = P->ncap[s];
                if ((int64_t)n1 + n2 > capg) {
                    bad = 1;
                    continue;
                }
                keys.clear();
                certificate_bridges(P->h_area0 + off, n1, P->h_area0 + off + capg - n2, n2, P->V[g], sc, keys);
                canonical_sort(keys);
                std::copy(keys.begin(), keys.end(), outk + slot[s]);
                nb[g] = (int64_t)keys.size();
            }
        });
        if (bad) return fail(BR_EINTERNAL, "batched: certificate counts exceed their region");
    }
    auto t2 = std::chrono::steady_clock::now();
    // graphs above the LDS limit: the plain path, with the same chunk size
    std::vector<std::vector<int32_t>> large_out(P->large.size());
    for (size_t k = 0; k < P->large.size(); k++) {
        const int32_t g = P->large[k];
        const int64_t E = h_edge_off[g + 1] - h_edge_off[g];
        const int32_t M = (int32_t)std::max<int64_t>(1, std::min<int64_t>((E + C - 1) / C, 1 << 20));
        large_out[k].resize(2 * (size_t)std::max(h_V[g] - 1, 1));
        int64_t n = 0;
        rc = br_bridges_find(c, d_edges + 2 * h_edge_off[g], E, h_V[g], M, large_out[k].data(),
                             std::max(h_V[g] - 1, 1), &n, st.stream);
        if (rc) return rc;
        nb[g] = n;
        large_out[k].resize(2 * (size_t)n);
    }
    // assemble in graph order
    h_bridge_off[0] = 0;
    for (int32_t g = 0; g < G; g++) h_bridge_off[g + 1] = h_bridge_off[g] + nb[g];
    const int64_t total = h_bridge_off[G];
    if (total <= cap) {
        for (int32_t s = 0; s < S; s++) {
            const int32_t g = P->small[s];
            int32_t* o = h_bridges + 2 * h_bridge_off[g];
            if (mode == 1) {
                const uint32_t* k = keys + P->h_sb[16 + 2 * s];
                for (int64_t i = 0; i < nb[g]; i++) {
                    o[2 * i] = (int32_t)(k[i] >> 16);
                    o[2 * i + 1] = (int32_t)(k[i] & 0xffffu);
                }
            } else {
                for (int64_t i = 0; i < nb[g]; i++) {
                    o[2 * i] = (int32_t)(outk[slot[s] + i] >> 32);
                    o[2 * i + 1] = (int32_t)(outk[slot[s] + i] & 0xffffffffu);
                }
            }
        }
        for (size_t k = 0; k < P->large.size(); k++)
            std::copy(large_out[k].begin(), large_out[k].end(), h_bridges + 2 * h_bridge_off[P->large[k]]);
        for (size_t k = 0; k < mid.size(); k++)
            std::copy(mid_out[k].begin(), mid_out[k].end(), h_bridges + 2 * h_bridge_off[mid[k]]);
    }
    auto t3 = std::chrono::steady_clock::now();
    if (c->profiling) {
        float ms = 0.f;
        if (hipEventElapsedTime(&ms, st.e0, st.e1) != hipSuccess) ms = 0.f;
        c->prof.ms_cert = ms;
        if (hipEventElapsedTime(&ms, st.k0, st.k1) != hipSuccess) ms = 0.f;   // clear + persistent kernel
        c->prof.ms_phase0 = ms;
        if (hipEventElapsedTime(&ms, st.k1, st.k2) != hipSuccess) ms = 0.f;   // combined bridge step (if any)
        c->prof.ms_bridge_dev = mode == 1 ? ms : 0.0;
        (void)hipGetLastError();
        c->prof.ms_merge = 0;
        c->prof.ms_d2h = 0;
    }
    c->prof.ms_dfs = std::chrono::duration<double, std::milli>(t2 - t1).count();
    c->prof.ms_canon = std::chrono::duration<double, std::milli>(t3 - t2).count();
    c->prof.ms_total = std::chrono::duration<double, std::milli>(t3 - t0).count();
    c->prof.rounds = C;
    c->prof.launches = 1;
    if (total > cap) return fail(BR_ECAP, "batched: %lld bridges, capacity %lld", (long long)total, (long long)cap);
    return BR_OK;
}

}  // namespace br

using namespace br;

extern "C" {

int32_t br_batched_max_v(void) { return batched_max_v_dev(); }
int32_t br_lds_max_v(void) { return batched_max_v_big(); }

int br_bridges_find_batched(br_ctx* c, const int32_t* d_edges, const int64_t* h_edge_off, const int32_t* h_V,
                            int32_t G, int32_t chunk_edges, int32_t* h_bridges, int64_t cap, int64_t* h_bridge_off,
                            void* stream) {
    if (!c || !h_edge_off || !h_V || !h_bridge_off || G < 0 || chunk_edges < 0 || cap < 0 || (cap > 0 && !h_bridges))
        return fail(BR_EINVAL, "br_bridges_find_batched: bad argument");
    if (h_edge_off[0] != 0) return fail(BR_EINVAL, "batched: offsets must start at 0");
    for (int32_t g = 0; g < G; g++) {
        if (h_edge_off[g + 1] < h_edge_off[g]) return fail(BR_EINVAL, "batched: offsets decrease at graph %d", g);
        if (h_V[g] < 1) return fail(BR_EINVAL, "batched: V[%d] = %d < 1", g, h_V[g]);
    }
    if (h_edge_off[G] > 0 && !d_edges) return fail(BR_EINVAL, "batched: null edge list");
    return batched_query(c, d_edges, h_edge_off, h_V, G, chunk_edges, h_bridges, cap, h_bridge_off, stream, false);
}

}  // extern "C"
