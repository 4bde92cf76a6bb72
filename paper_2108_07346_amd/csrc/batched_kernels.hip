// Batched certificates for many small graphs in one persistent launch (and two
// more for those with long lists).
//
// Work items are (graph, chunk) pairs: graph g's edge list is split into M_g
// chunks exactly as in the paper's phase tree (Section III), and the items are
// handed out largest-first from a device queue.  A workgroup certifies one
// chunk (Algorithm 2) with the whole union-find state in LDS, then takes part
// in the graph's merge tree: the merge of nodes i and i + 2^(q-1) in round q
// is done by whichever workgroup finishes the second of the two (an arrival
// counter per merge), re-running the certificate on the union of the two
// certificates, again in LDS.  Node 0's region of each graph ends up holding
// the graph's certificate: F from the front, F' from the back.
//
// LDS union-find: one 32-bit word per vertex, low half = x - parent in F,
// high half = x - parent in F' (0 = root; V <= 65,536 keeps both in 16 bits).
// Two instances: graphs up to 4,096 vertices (three workgroups per CU) and
// graphs up to 40,944 vertices (the whole LDS of a CU, one workgroup; only with
// the search on the host, else those are one query over their union).
//
// Graphs with many edges per vertex are not split at all: every chunk would hook
// its own forests and every merge hook them again, in a chain that the largest
// graph's chunks set the length of.  One item takes rows spread over the list,
// about 4V to 6V edges, after which nearly every other edge lies inside a
// component of F'; a second launch sends the rest past that state in independent
// runs, and a third offers what those kept to it (launch_batched_long).
// Hooking is a 32-bit LDS compare-and-swap that changes one half; a swap that
// fails because the other half moved is simply retried.  The larger root is
// hooked under the smaller representative, so chains decrease and the loop
// ends (see cert_kernels.hip for the argument).

#include <hip/hip_runtime.h>

#include "device_util.hpp"
#include "internal.hpp"
#include "lds_union_find.hpp"

namespace br {

namespace {

constexpr int kBB = 512;          // threads per workgroup
constexpr int kMaxV = 4096;       // vertices per graph of the small kernel
// the large kernel: the whole 160 KB of a CU's LDS for one graph's state, less
// the counters (the offsets stay 16-bit: V <= 65,536)
constexpr int kMaxVBig = (160 * 1024 - 64) / 4;

// Staged = true: a merge re-runs the certificate on X_i u X_j into a fresh
// state, staging the result in LDS before writing node i's region back (the
// small kernel).  Staged = false: a merge rebuilds node i's state from its
// own certificate (F's edges into F, F''s into F' -- all accepted, nothing
// written) and streams X_j in, appending what is accepted to node i's region
// after its edges (the same certificate as the state-carrying merge; no
// stage, so the state can take all of LDS).
template <int MaxV, bool Staged>
struct LdsState {
    static constexpr int kStage = Staged ? 2 * (MaxV - 1) : 1;
    uint32_t q[MaxV];             // packed F / F' offsets
    uint32_t stage[kStage];       // merged certificate: (u | v << 16), F from front, F' from back
    uint32_t n12;                 // edges of the current certificate: F in the low half, F' in the high
                                  // (each a forest count, at most V - 1 < 2^16, so no carry)
    int32_t item, last, errv;
};

__device__ __forceinline__ int64_t part_lo(int64_t E, int64_t M, int64_t i) { return i * (E / M) + (i * (E % M)) / M; }

}  // namespace



namespace {

// Certify edges [t0, t1) of graph g (ids < V) into an empty LDS state and write
// the accepted edges to node region (off, cap).  Counts go to S.n12.
// Each thread takes 2 kU edges per step and the next step's edges are loaded
// before the current ones are offered, so that enough loads are in flight to
// cover HBM latency while the LDS work proceeds.
constexpr int kU = 4;

typedef int edge2 __attribute__((ext_vector_type(4), aligned(8)));   // two edges, 8-byte aligned

// The edges a workgroup certifies: [t0, t1), or of those (stride > 1) the rows
// of kLongRow that are multiples of stride, counted as one sequence of n.  Rows
// are no longer than four 128-byte lines: a list sorted by vertex shows as many
// of its vertices as the sample can hold.
struct Seq {
    int64_t t0, t1, n;
    int32_t stride;
    __device__ Seq(int64_t a, int64_t b, int32_t s) : t0(a), t1(b), n(b - a), stride(s) {
        if (s > 1) {
            const int64_t rows = (b - a + kLongRow - 1) / kLongRow;
            n = (rows + s - 1) / s * kLongRow;
        }
    }
    __device__ int64_t at(int64_t r) const { return stride > 1 ? t0 + r / kLongRow * stride * kLongRow + r % kLongRow : t0 + r; }
};

// The edges of a step: kU pairs per thread.  The result tells which of them exist.
__device__ __forceinline__ uint32_t load_step(const BatchDev& B, const Seq& Q, int64_t rel, int2 (&e)[2 * kU]) {
    const int64_t r0 = rel + 2 * threadIdx.x;
    if (rel + 2 * kBB * kU <= (Q.stride > 1 ? Q.n - kLongRow : Q.n)) {      // a whole step (the same for every thread)
#pragma unroll
        for (int j = 0; j < kU; j++) {
            const edge2 w = *reinterpret_cast<const edge2*>(B.edges + Q.at(r0 + j * 2 * kBB));
            e[2 * j] = make_int2(w.x, w.y);
            e[2 * j + 1] = make_int2(w.z, w.w);
        }
        return (1u << 2 * kU) - 1u;
    }
    uint32_t ok = 0;
#pragma unroll
    for (int j = 0; j < 2 * kU; j++) {
        const int64_t r = r0 + (j >> 1) * 2 * kBB + (j & 1), i = Q.at(r);
        e[j] = make_int2(0, 0);
        if (r < Q.n && i < Q.t1) {
            e[j] = B.edges[i];
            ok |= 1u << j;
        }
    }
    return ok;
}

// What bounds it: instructions.  Most edges of a dense chunk end at the shared
// parent in F' (two 16-bit LDS reads and a compare, which rejects the edge in F
// too); loaded two to a 16-byte load and tested without 64-bit index arithmetic
// per edge, they leave the time to the ones that search.
template <class LS>
__device__ void certify_chunk(LS& S, const BatchDev& B, const Seq& Q, uint32_t V, int64_t off, int64_t cap) {
    for (uint32_t x = threadIdx.x; x < V; x += kBB) S.q[x] = 0;
    if (threadIdx.x == 0) S.n12 = 0;
    __syncthreads();
    // compress after the first 2V and 8V edges (dense chunks are then mostly
    // rejected by the shared-parent test)
    int64_t next_cmp = 2 * (int64_t)V;
    constexpr int64_t kStep = (int64_t)kBB * 2 * kU;
    int2 cur[2 * kU], nxt[2 * kU];
    uint32_t ok = load_step(B, Q, 0, cur), nok = 0;
    const lds_half* h2 = reinterpret_cast<const lds_half*>(S.q) + 1;     // x - parent in F' at h2[2 x]
    for (int64_t rel = 0; rel < Q.n; rel += kStep) {
        if (rel >= next_cmp) {
            __syncthreads();
            lcompress(S.q, V);
            __syncthreads();
            next_cmp = next_cmp == 2 * (int64_t)V ? 8 * (int64_t)V : INT64_MAX;
        }
        nok = load_step(B, Q, rel + kStep, nxt);
        if constexpr (LS::kStage >= kBB * 2 * kU) {
            // Where the stage area is free (it only serves merges), each
            // wavefront first applies the shared-parent test to all of its
            // 2 kU x 64 edges and packs the ones the test cannot reject into a
            // list of its own there; those are then offered 64 at a time, so
            // that the searches of a few lanes no longer hold a whole
            // wavefront (in a dense chunk most edges are rejected by the test).
            uint32_t* wl = S.stage + (threadIdx.x / 64) * (128 * kU);
            uint32_t nh = 0;
#pragma unroll
            for (int j = 0; j < 2 * kU; j++) {
                const uint32_t x = (uint32_t)cur[j].x, y = (uint32_t)cur[j].y;
                bool hard = false;
                if (ok >> j & 1u) {
                    if (max(x, y) < V) hard = x - h2[2 * x] != y - h2[2 * y];
                    else atomicOr(B.err, 1u);
                }
                const uint64_t m = __ballot(hard);
                if (m) {
                    if (hard) wl[nh + lane_rank(m)] = x | (y << 16);
                    nh += (uint32_t)__popcll(m);
                }
            }
            __builtin_amdgcn_wave_barrier();     // the list, written by the wavefront's lanes, is read back by them
            for (uint32_t k0 = 0; k0 < nh; k0 += 64) {
                const uint32_t k = k0 + __lane_id();
                bool a1 = false, a2 = false;
                int2 e = make_int2(0, 0);
                if (k < nh) {
                    const uint32_t w = wl[k];
                    e = make_int2((int32_t)(w & 0xffffu), (int32_t)(w >> 16));
                    loffer(S.q, (uint32_t)e.x, (uint32_t)e.y, a1, a2);
                }
                uint32_t p1, p2;
                reserve2(&S.n12, a1, a2, p1, p2);
                if (a1) { if (p1 < cap) B.cert[off + p1] = e; else atomicOr(B.err, 2u); }
                if (a2) { if (p2 < cap) B.cert[off + cap - 1 - p2] = e; else atomicOr(B.err, 2u); }
            }
            __builtin_amdgcn_wave_barrier();     // every lane's reads of the list before the next step's writes
        } else {
#pragma unroll
            for (int j = 0; j < 2 * kU; j++) {
                const int2 e = cur[j];
                bool a1 = false, a2 = false;
                if (ok >> j & 1u) {
                    if ((uint32_t)e.x < V && (uint32_t)e.y < V) loffer(S.q, (uint32_t)e.x, (uint32_t)e.y, a1, a2);
                    else atomicOr(B.err, 1u);
                }
                uint32_t p1, p2;
                reserve2(&S.n12, a1, a2, p1, p2);
                if (a1) { if (p1 < cap) B.cert[off + p1] = e; else atomicOr(B.err, 2u); }
                if (a2) { if (p2 < cap) B.cert[off + cap - 1 - p2] = e; else atomicOr(B.err, 2u); }
            }
        }
#pragma unroll
        for (int j = 0; j < 2 * kU; j++) cur[j] = nxt[j];
        ok = nok;
    }
    __syncthreads();
}

// Offer the certificate stored in node region (off, cap) with counts (n1, n2)
// to the LDS state, staging accepted edges in S.stage.
template <class LS>
__device__ void offer_region(LS& S, const BatchDev& B, int64_t off, int64_t cap, uint32_t n1, uint32_t n2,
                             uint32_t maxv) {
    constexpr int kStage = LS::kStage;
    const int64_t total = (int64_t)n1 + n2;
    for (int64_t base = 0; base < total; base += kBB) {
        const int64_t k = base + threadIdx.x;
        bool a1 = false, a2 = false;
        int2 e = make_int2(0, 0);
        if (k < total) {
            const uint64_t r = __hip_atomic_load(reinterpret_cast<const uint64_t*>(B.cert + (k < n1 ? off + k : off + cap - n2 + (k - n1))),
                                                 __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            e = make_int2((int32_t)(uint32_t)r, (int32_t)(uint32_t)(r >> 32));
            if ((uint32_t)e.x < maxv && (uint32_t)e.y < maxv) loffer(S.q, (uint32_t)e.x, (uint32_t)e.y, a1, a2);
            else atomicOr(B.err, 2u);
        }
        const uint32_t w = (uint32_t)e.x | ((uint32_t)e.y << 16);
        uint32_t p1, p2;
        reserve2(&S.n12, a1, a2, p1, p2);
        if (a1) { if (p1 < kStage) S.stage[p1] = w; else atomicOr(B.err, 2u); }
        if (a2) { if (p2 < kStage) S.stage[kStage - 1 - p2] = w; else atomicOr(B.err, 2u); }
    }
}

__device__ __forceinline__ int2 region_edge(const BatchDev& B, int64_t off, int64_t cap, uint32_t n1, uint32_t n2,
                                            int64_t k) {
    const uint64_t r = __hip_atomic_load(reinterpret_cast<const uint64_t*>(B.cert + (k < n1 ? off + k : off + cap - n2 + (k - n1))),
                                         __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return make_int2((int32_t)(uint32_t)r, (int32_t)(uint32_t)(r >> 32));
}

// Node i's state from its certificate in (off, cap): F's edges hooked in F,
// then (after a barrier) F''s in F'.  Each set is a forest, so every edge is
// accepted whatever the order; nothing is written.
template <class LS>
__device__ void rebuild_state(LS& S, const BatchDev& B, int64_t off, int64_t cap, uint32_t n1, uint32_t n2,
                              uint32_t V) {
    for (int64_t k = threadIdx.x; k < n1; k += kBB) {
        const int2 e = region_edge(B, off, cap, n1, n2, k);
        if ((uint32_t)e.x < V && (uint32_t)e.y < V) (void)lunite<0>(S.q, (uint32_t)e.x, (uint32_t)e.y);
        else atomicOr(B.err, 2u);
    }
    __syncthreads();
    for (int64_t k = (int64_t)n1 + threadIdx.x; k < (int64_t)n1 + n2; k += kBB) {
        const int2 e = region_edge(B, off, cap, n1, n2, k);
        if ((uint32_t)e.x < V && (uint32_t)e.y < V) (void)lunite<1>(S.q, (uint32_t)e.x, (uint32_t)e.y);
        else atomicOr(B.err, 2u);
    }
}

// The certificate in (offj, capj) offered to the state; accepted edges are
// appended to region (offi, capi) after the edges S.n12 already counts.
template <class LS>
__device__ void offer_region_append(LS& S, const BatchDev& B, int64_t offj, int64_t capj, uint32_t n1, uint32_t n2,
                                    uint32_t V, int64_t offi, int64_t capi) {
    const int64_t total = (int64_t)n1 + n2;
    for (int64_t base = 0; base < total; base += kBB) {
        const int64_t k = base + threadIdx.x;
        bool a1 = false, a2 = false;
        int2 e = make_int2(0, 0);
        if (k < total) {
            e = region_edge(B, offj, capj, n1, n2, k);
            if ((uint32_t)e.x < V && (uint32_t)e.y < V) loffer(S.q, (uint32_t)e.x, (uint32_t)e.y, a1, a2);
            else atomicOr(B.err, 2u);
        }
        uint32_t p1, p2;
        reserve2(&S.n12, a1, a2, p1, p2);
        if (a1) { if (p1 < capi) B.cert[offi + p1] = e; else atomicOr(B.err, 2u); }
        if (a2) { if (p2 < capi) B.cert[offi + capi - 1 - p2] = e; else atomicOr(B.err, 2u); }
    }
}

}  // namespace

namespace {

// parent in H's forest (roots of F' as vertices; H may be read while it changes)
__device__ __forceinline__ uint32_t c_find(uint32_t* par, uint32_t x) {
    for (uint32_t p = par[x]; p != x; p = par[x]) {
        const uint32_t g = par[p];
        par[x] = g;
        x = g;
    }
    return x;
}
__device__ __forceinline__ bool c_unite(uint32_t* par, uint32_t a, uint32_t b) {
    for (;;) {
        a = c_find(par, a);
        b = c_find(par, b);
        if (a == b) return false;
        if (a < b) { const uint32_t t = a; a = b; b = t; }
        if (atomicCAS(&par[a], a, b) == a) return true;
    }
}

// Bridges of the graph whose certificate is in region (off, cap) and whose
// union-find state is in S.q, by contracting the components of F' (contract.hpp
// has the reason): the edges of F that cross components are all bridges if they
// form a forest; otherwise the graph goes to the list of those the second kernel
// roots and numbers.  Everything stays in the workgroup's LDS: the crossing
// edges in the stage, their forest, then the sorted keys in the state's place.
template <class LS>
__device__ void finish_graph(LS& S, const BatchDev& B, int32_t g, uint32_t V, int64_t off, uint32_t n1) {
    uint32_t* he = S.stage;                      // [n1] a | b << 16, roots of F'
    uint16_t* hk = reinterpret_cast<uint16_t*>(S.stage + kMaxV);     // [n1] place in F
    uint32_t* ctr = S.stage + kMaxV + kMaxV / 2;  // 0: crossing edges, 1: one of them closes a cycle, 2: keys' base
    // F' alone: nothing here asks for F's roots, and a path or a tree in vertex order
    // leaves chains of up to V there and none in F' (3 paths of 4,000 vertices: 125 us
    // for the kernel with both compressed, 109 so)
    for (uint32_t x = threadIdx.x; x < V; x += kBB) {
        lds_half* h = reinterpret_cast<lds_half*>(S.q) + 1;
        uint32_t r = x - h[2 * x];
        for (uint32_t d = h[2 * r]; d; d = h[2 * r]) r -= d;
        h[2 * x] = (uint16_t)(x - r);
    }
    if (threadIdx.x < 3) ctr[threadIdx.x] = 0;
    __syncthreads();
    for (uint32_t k = threadIdx.x; k < n1; k += kBB) {
        const int2 e = region_edge(B, off, 0, n1, 0, k);
        const uint32_t a = (uint32_t)e.x - (S.q[e.x] >> 16), b = (uint32_t)e.y - (S.q[e.y] >> 16);
        if (a != b) {
            const uint32_t p = atomicAdd(&ctr[0], 1u);
            he[p] = a | b << 16;
            hk[p] = (uint16_t)k;
        }
    }
    __syncthreads();
    const uint32_t m = ctr[0];
    uint32_t* par = S.q;
    for (uint32_t x = threadIdx.x; x < V; x += kBB) par[x] = x;
    __syncthreads();
    for (uint32_t j = threadIdx.x; j < m; j += kBB)
        if (!c_unite(par, he[j] & 0xffffu, he[j] >> 16)) ctr[1] = 1;
    __syncthreads();
    if (ctr[1]) {
        if (threadIdx.x == 0) {
            const bool a = (int32_t)V <= B.split_v;
            (a ? B.list_a : B.list_b)[atomicAdd(&B.out_hdr[a ? 2 : 3], 1u)] = g;
        }
        __syncthreads();
        return;
    }
    // keys, sorted (bitonic), and their place in the output
    uint32_t* key = S.q;
    uint32_t P = 1;
    while (P < m) P <<= 1;
    for (uint32_t j = threadIdx.x; j < P; j += kBB) {
        uint32_t w = 0xffffffffu;
        if (j < m) {
            const int2 e = region_edge(B, off, 0, n1, 0, hk[j]);
            w = (uint32_t)min(e.x, e.y) << 16 | (uint32_t)max(e.x, e.y);
        }
        key[j] = w;
    }
    __syncthreads();
    for (uint32_t k = 2; k <= P; k <<= 1)
        for (uint32_t j = k >> 1; j > 0; j >>= 1) {
            for (uint32_t i = threadIdx.x; i < P; i += kBB) {
                const uint32_t q = i ^ j;
                if (q > i) {
                    const uint32_t x = key[i], y = key[q];
                    if (((i & k) == 0) == (x > y)) { key[i] = y; key[q] = x; }
                }
            }
            __syncthreads();
        }
    if (threadIdx.x == 0) {
        ctr[2] = m ? atomicAdd(B.out_hdr, m) : 0u;
        B.out_hdr[16 + 2 * g] = ctr[2];
        B.out_hdr[16 + 2 * g + 1] = m;
    }
    __syncthreads();
    for (uint32_t j = threadIdx.x; j < m; j += kBB) B.out_keys[ctr[2] + j] = key[j];
    __syncthreads();
}

}  // namespace

template <int MaxV, bool Staged>
__global__ void __launch_bounds__(kBB) k_batched(BatchDev B) {
    using LS = LdsState<MaxV, Staged>;
    constexpr int kStage = LS::kStage;
    __shared__ LS S;
    for (;;) {
        if (threadIdx.x == 0) S.item = (int32_t)atomicAdd(B.queue, 1u);
        __syncthreads();
        const int64_t it = S.item;
        if (it >= B.n_items) break;
        const int64_t code = B.items[it];
        const int32_t g = (int32_t)(code >> 20);
        int64_t node = code & ((1 << 20) - 1);
        const int64_t Mg = B.Mg[g];
        const uint32_t V = (uint32_t)B.V[g];
        const int64_t e0 = B.eoff[2 * g], Eg = B.eoff[2 * g + 1] - e0;
        const int64_t rb = B.rbase[g];
        auto nidx = [&](int64_t k) { return k ? rb + k - 1 : (int64_t)g; };
        // phase 0: chunk `node` of graph g
        const int32_t stride = Staged && B.stride ? B.stride[g] : 0;
        certify_chunk(S, B, Seq(e0 + part_lo(Eg, Mg, node), e0 + part_lo(Eg, Mg, node + 1), max(stride, 1)), V,
                      B.noff[nidx(node)], B.ncap[nidx(node)]);
        uint32_t n1 = S.n12 & 0xffffu, n2 = S.n12 >> 16;
        if (stride > 0) {
            // a long graph: its state goes to memory
            lcompress(S.q, V);
            __syncthreads();
            const int64_t vb = B.vbase[g];
            for (uint32_t x = threadIdx.x; x < V; x += kBB) B.stq[vb + x] = S.q[x];
            if (threadIdx.x == 0) {
                B.ncnt[2 * g] = n1;
                B.ncnt[2 * g + 1] = n2;
            }
            __syncthreads();
            continue;
        }
        // merge rounds: climb while this workgroup is the second of a pair to finish
        int64_t step = 1, level = 0, cb = B.cbase[g];
        for (;;) {
            if (threadIdx.x == 0) {
                B.ncnt[2 * nidx(node)] = n1;
                B.ncnt[2 * nidx(node) + 1] = n2;
            }
            if (step >= Mg) {                               // node 0 holds the graph's certificate
                // the LDS state encodes its F: publish the roots of F's trees
                const int64_t vb = B.vbase[g];
                for (uint32_t x = threadIdx.x; x < V; x += kBB) B.rootw[vb + x] = (S.q[x] & 0xffffu) ? 1u : 0u;
                if constexpr (Staged)
                    if (B.out_hdr) {
                        __syncthreads();
                        finish_graph(S, B, g, V, B.noff[g], n1);
                    }
                break;
            }
            const int64_t i = node & ~(2 * step - 1);       // left node of this round's pair
            const int64_t j = i + step;
            if (j >= Mg) {                                  // no partner: pass through
                node = i;
                step *= 2;
                level++;
                continue;
            }
            // publish this node's certificate: the barrier orders every
            // thread's stores before thread 0's device-scope release (which
            // writes the XCD's L2 back), then one arrival per workgroup
            __syncthreads();
            if (threadIdx.x == 0) {
                __threadfence();
                const uint32_t prev = atomicAdd(&B.arrive[cb + level * ((Mg + 1) / 2) + (i >> (level + 1))], 1u);
                S.last = prev == 1u;
                if (S.last) __threadfence();                // acquire the partner's certificate
            }
            __syncthreads();
            if (!S.last) break;                             // the partner will merge
            // merge: Certificate(X_i u X_j), staged in LDS, written back to node i
            for (uint32_t x = threadIdx.x; x < V; x += kBB) S.q[x] = 0;
            if (threadIdx.x == 0) S.n12 = 0;
            __syncthreads();
            const uint32_t ai1 = __hip_atomic_load(&B.ncnt[2 * nidx(i)], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const uint32_t ai2 = __hip_atomic_load(&B.ncnt[2 * nidx(i) + 1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const uint32_t aj1 = __hip_atomic_load(&B.ncnt[2 * nidx(j)], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const uint32_t aj2 = __hip_atomic_load(&B.ncnt[2 * nidx(j) + 1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const int64_t offi = B.noff[nidx(i)], capi = B.ncap[nidx(i)];
            const int64_t offj = B.noff[nidx(j)], capj = B.ncap[nidx(j)];
            const uint32_t ci1 = min(ai1, (uint32_t)capi), ci2 = min(ai2, (uint32_t)capi - ci1);
            const uint32_t cj1 = min(aj1, (uint32_t)capj), cj2 = min(aj2, (uint32_t)capj - cj1);
            if constexpr (Staged) {
                offer_region(S, B, offi, capi, ci1, ci2, (uint32_t)MaxV);
                offer_region(S, B, offj, capj, cj1, cj2, (uint32_t)MaxV);
                __syncthreads();
                n1 = min(S.n12 & 0xffffu, (uint32_t)kStage);
                n2 = min(S.n12 >> 16, (uint32_t)kStage - n1);
                if ((int64_t)n1 + n2 > capi) {
                    if (threadIdx.x == 0) atomicOr(B.err, 2u);
                    n1 = 0;
                    n2 = 0;
                }
                for (uint32_t k = threadIdx.x; k < n1 + n2; k += kBB) {
                    const uint32_t w = k < n1 ? S.stage[k] : S.stage[kStage - n2 + (k - n1)];
                    const int64_t pos = k < n1 ? offi + k : offi + capi - n2 + (k - n1);
                    B.cert[pos] = make_int2((int32_t)(w & 0xffffu), (int32_t)(w >> 16));
                }
            } else {
                rebuild_state(S, B, offi, capi, ci1, ci2, V);
                if (threadIdx.x == 0) S.n12 = ci1 | (ci2 << 16);
                __syncthreads();
                offer_region_append(S, B, offj, capj, cj1, cj2, V, offi, capi);
                __syncthreads();
                n1 = S.n12 & 0xffffu;
                n2 = S.n12 >> 16;
                if ((int64_t)n1 + n2 > capi && threadIdx.x == 0) atomicOr(B.err, 2u);
            }
            __syncthreads();
            node = i;
            step *= 2;
            level++;
        }
        __syncthreads();
    }
}

namespace {

// A run of a long graph's list (all but the rows its first item took) on a copy
// of the state after those rows.  An edge whose ends have the same parent in F'
// is rejected by both forests: two LDS reads, which nearly every edge ends at.
// The others go through the searches a full wavefront at a time, from a list
// that each wavefront keeps; those that either forest takes go to the graph's
// list.  A run keeps at most what its forests still had room for, so the lists
// are bounded also where the first rows told nothing.
// What bounds it: HBM.  4,096 graphs of 64 to 4,096 vertices (1.4 GB, of which
// the 375 long graphs hold 0.94): these runs 165 us (5.7 TB/s) and k_batch_finish
// 22 us, k_batched's part 310 us; all in chunks and merges, k_batched took 603 us.
__global__ void __launch_bounds__(kBB) k_batch_runs(BatchDev B) {
    constexpr int kW = kBB / 64, kCap = 128, kP = 4;
    __shared__ uint32_t q[kMaxV];
    __shared__ uint32_t lists[kW][kCap];
    const int64_t code = B.fitems[blockIdx.x];
    const int32_t g = (int32_t)(code >> 32);
    const uint32_t V = (uint32_t)B.V[g], stride = (uint32_t)B.stride[g];
    const int64_t e0 = B.eoff[2 * g], vb = B.vbase[g], sb = B.sbase[g];
    const int64_t i0 = (int64_t)(uint32_t)code * kLongRun, i1 = min(i0 + kLongRun, B.eoff[2 * g + 1] - e0);
    const uint32_t row0 = (uint32_t)(i0 / kLongRow);
    for (uint32_t x = threadIdx.x; x < V; x += kBB) q[x] = B.stq[vb + x];
    __syncthreads();
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const lds_half* par = reinterpret_cast<const lds_half*>(q) + 1;
    uint32_t* wl = lists[wave];
    uint32_t n = 0;
    auto offer = [&](uint32_t first, bool mine) {
        bool a1 = false, a2 = false;
        uint32_t w = 0;
        if (mine) {
            w = wl[first + lane];
            loffer(q, w & 0xffffu, w >> 16, a1, a2);
        }
        const uint64_t m = __ballot(a1 || a2);
        if (m) {
            uint32_t at = 0;
            if (lane == 0) at = atomicAdd(&B.scnt[g], (uint32_t)__popcll(m));
            at = __shfl(at, 0) + lane_rank(m);
            if (a1 || a2) {
                if (sb + at < B.sbase[g + 1]) B.surv[sb + at] = w;
                else atomicOr(B.err, 2u);
            }
        }
    };
    const uint32_t n_units = (uint32_t)((i1 - i0 + 127) >> 7);         // 128 edges: two rows
    for (uint32_t u = wave; u < n_units; u += kW * kP) {
        int2 e[2 * kP];
        uint32_t ok = 0;
#pragma unroll
        for (int j = 0; j < kP; j++) {
            const uint32_t uu = u + j * kW;
            const int64_t i = i0 + uu * 128 + 2 * lane;
            const uint32_t rem = (row0 + 2 * uu) % stride;             // the same for the wavefront
            e[2 * j] = e[2 * j + 1] = make_int2(0, 0);
            if (i < i1 && rem != (lane < 32 ? 0u : stride - 1)) {
                if (i + 1 < i1) {
                    const edge2 w = *reinterpret_cast<const edge2*>(B.edges + e0 + i);
                    e[2 * j] = make_int2(w.x, w.y);
                    e[2 * j + 1] = make_int2(w.z, w.w);
                    ok |= 3u << (2 * j);
                } else {
                    e[2 * j] = B.edges[e0 + i];
                    ok |= 1u << (2 * j);
                }
            }
        }
#pragma unroll
        for (int j = 0; j < 2 * kP; j++) {
            const uint32_t x = (uint32_t)e[j].x, y = (uint32_t)e[j].y;
            bool hard = false;
            if (ok >> j & 1u) {
                if (max(x, y) < V) hard = x - par[2 * x] != y - par[2 * y];
                else atomicOr(B.err, 1u);
            }
            const uint64_t m = __ballot(hard);
            if (m) {
                if (hard) wl[n + lane_rank(m)] = x | y << 16;
                n += (uint32_t)__popcll(m);
                __builtin_amdgcn_wave_barrier();
                if (n >= 64) {
                    n -= 64;
                    offer(n, true);
                    __builtin_amdgcn_wave_barrier();
                }
            }
        }
    }
    if (n) offer(0, lane < n);
}

// The edges that the runs kept offered to the state after the first rows, and
// the graph's final step.
__global__ void __launch_bounds__(kBB) k_batch_finish(BatchDev B) {
    using LS = LdsState<kMaxV, true>;
    __shared__ LS S;
    const int32_t g = B.longs[blockIdx.x];
    const uint32_t V = (uint32_t)B.V[g];
    const int64_t vb = B.vbase[g], sb = B.sbase[g], off = B.noff[g], cap = B.ncap[g];
    for (uint32_t x = threadIdx.x; x < V; x += kBB) S.q[x] = B.stq[vb + x];
    if (threadIdx.x == 0) S.n12 = B.ncnt[2 * g] | B.ncnt[2 * g + 1] << 16;
    __syncthreads();
    const uint32_t ns = (uint32_t)min((int64_t)B.scnt[g], B.sbase[g + 1] - sb);
    uint32_t next = threadIdx.x < ns ? B.surv[sb + threadIdx.x] : 0u;
    for (uint32_t base = 0; base < ns; base += kBB) {
        const uint32_t k = base + threadIdx.x, w = next;
        if (k + kBB < ns) next = B.surv[sb + k + kBB];
        bool a1 = false, a2 = false;
        if (k < ns) loffer(S.q, w & 0xffffu, w >> 16, a1, a2);
        uint32_t p1, p2;
        reserve2(&S.n12, a1, a2, p1, p2);
        const int2 e = make_int2((int32_t)(w & 0xffffu), (int32_t)(w >> 16));
        if (a1) { if (p1 < cap) B.cert[off + p1] = e; else atomicOr(B.err, 2u); }
        if (a2) { if (p2 < cap) B.cert[off + cap - 1 - p2] = e; else atomicOr(B.err, 2u); }
    }
    __syncthreads();
    const uint32_t n1 = S.n12 & 0xffffu, n2 = S.n12 >> 16;
    if (threadIdx.x == 0) {
        if ((int64_t)n1 + n2 > cap) atomicOr(B.err, 2u);
        B.ncnt[2 * g] = n1;
        B.ncnt[2 * g + 1] = n2;
    }
    for (uint32_t x = threadIdx.x; x < V; x += kBB) B.rootw[vb + x] = (S.q[x] & 0xffffu) ? 1u : 0u;
    __syncthreads();
    if (B.out_hdr) finish_graph(S, B, g, V, off, n1);
}

}  // namespace

void launch_batched_long(const BatchDev& B, hipStream_t s) {
    if (B.n_long <= 0) return;
    if (B.n_fitems > 0) hipLaunchKernelGGL(k_batch_runs, dim3((unsigned)B.n_fitems), dim3(kBB), 0, s, B);
    hipLaunchKernelGGL(k_batch_finish, dim3((unsigned)B.n_long), dim3(kBB), 0, s, B);
}

void launch_batched(const BatchDev& B, int blocks, hipStream_t s, bool big) {
    if (big) hipLaunchKernelGGL((k_batched<kMaxVBig, false>), dim3(blocks), dim3(kBB), 0, s, B);
    else hipLaunchKernelGGL((k_batched<kMaxV, true>), dim3(blocks), dim3(kBB), 0, s, B);
}

int32_t batched_max_v_dev() { return kMaxV; }
int32_t batched_max_v_big() { return kMaxVBig; }

namespace {
// Gather of several device edge lists into one packed buffer: item x copies
// items[x].n edges from items[x].src to dst + items[x].at, the blocks of
// column y taking runs y, y + gridDim.y, ... of kGatherRun edges.
constexpr int64_t kGatherRun = 16384;
__global__ void __launch_bounds__(256) k_gather_edges(const GatherItem* items, int2* dst) {
    const GatherItem it = items[blockIdx.x];
    const int2* src = reinterpret_cast<const int2*>(it.src);
    for (int64_t lo = blockIdx.y * kGatherRun; lo < it.n; lo += (int64_t)gridDim.y * kGatherRun) {
        const int64_t hi = min(lo + kGatherRun, it.n);
        for (int64_t k = lo + threadIdx.x; k < hi; k += 256) dst[it.at + k] = src[k];
    }
}
}  // namespace

void launch_gather_edges(const GatherItem* d_items, int32_t n, int64_t max_edges, int32_t* dst, hipStream_t s) {
    if (n <= 0 || max_edges <= 0) return;
    const int64_t runs = std::min<int64_t>((max_edges + kGatherRun - 1) / kGatherRun, 1024);
    hipLaunchKernelGGL(k_gather_edges, dim3((unsigned)n, (unsigned)runs), dim3(256), 0, s, d_items,
                       reinterpret_cast<int2*>(dst));
}

namespace {
__global__ void __launch_bounds__(256) k_union_edges(const UnionItem* items, int32_t row, int2* dst) {
    const UnionItem it = items[blockIdx.x];
    const int2* src = reinterpret_cast<const int2*>(it.src);
    for (int64_t lo = blockIdx.y * kGatherRun; lo < it.n; lo += (int64_t)gridDim.y * kGatherRun) {
        const int64_t hi = min(lo + kGatherRun, it.n);
        for (int64_t k = lo + threadIdx.x; k < hi; k += 256) {
            const int2 e = src[k];
            const bool ok = (uint32_t)e.x < (uint32_t)it.V && (uint32_t)e.y < (uint32_t)it.V;
            dst[it.at + k] = ok ? make_int2(e.x + it.base, e.y + it.base) : make_int2(-1, -1);
        }
    }
    const int64_t end = (it.n + row - 1) / row * row;
    if (blockIdx.y == 0)
        for (int64_t k = it.n + threadIdx.x; k < end; k += 256) dst[it.at + k] = make_int2(it.base, it.base);
}
}  // namespace

void launch_union_edges(const UnionItem* d_items, int32_t n, int64_t max_edges, int32_t row, int32_t* dst, hipStream_t s) {
    if (n <= 0 || max_edges <= 0) return;
    const int64_t runs = std::min<int64_t>((max_edges + kGatherRun - 1) / kGatherRun, 1024);
    hipLaunchKernelGGL(k_union_edges, dim3((unsigned)n, (unsigned)runs), dim3(256), 0, s, d_items, row,
                       reinterpret_cast<int2*>(dst));
}

int32_t batched_blocks_per_cu() { return 3; }
// workgroups of the small kernel that fit one CU's LDS together
int32_t batched_max_blocks_per_cu() {
    return std::max<int32_t>(1, (int32_t)((160 * 1024) / sizeof(LdsState<kMaxV, true>)));
}

}  // namespace br
