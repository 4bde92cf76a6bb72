// The contracted certificate H and its bridges, by one workgroup (included by
// .hip sources only).
//
// An edge of F' was rejected by F, so F connects its endpoints without it:
// they are joined by two edge-disjoint paths and share a 2-edge-connected
// class.  Contracting every component of F' to one vertex therefore keeps the
// bridges and the classes of the certificate.  What remains are the edges of F
// that cross components (H): on a dense graph the pendant vertices, the edges
// between clusters and little else.  If H is a forest, all its edges are
// bridges.  Otherwise its hanging trees are stripped leaf by leaf (bridges
// again) and the rest, if it has at most kCoreV vertices, goes through the
// subtree test of small_bridges.hpp.
#pragma once

#include <hip/hip_runtime.h>

#include "internal.hpp"
#include "small_bridges.hpp"

namespace br {

constexpr int kCoreV = 4096;
constexpr int kSolveT = 1024;
constexpr int kPeelRounds = 48;

struct SolveLds {
    union {
        struct {
            uint32_t e[kMaxCross];          // H's edges, a | b << 16
            uint32_t par[kMaxCross + 1];    // parent in H's forest; then degree << 16 | xor of the incident edges; then new ids
        } h;
        SmallLds<kCoreV, kSolveT> small;
    };
    uint32_t tree[kMaxCross / 32];          // edge of H's forest
    uint32_t gone[kMaxCross / 32];          // edge stripped as a bridge
    uint32_t nnon, nout, ncore, nct, ncn, nuni, more;
};

__device__ __forceinline__ uint32_t h_find(uint32_t* par, uint32_t x) {
    for (;;) {
        const uint32_t p = par[x];
        if (p == x) return x;
        const uint32_t g = par[p];
        if (g == p) return p;
        par[x] = g;
        x = g;
    }
}

__device__ __forceinline__ bool h_unite(uint32_t* par, uint32_t a, uint32_t b) {
    for (;;) {
        a = h_find(par, a);
        b = h_find(par, b);
        if (a == b) return false;
        if (a < b) { const uint32_t t = a; a = b; b = t; }
        if (atomicCAS(&par[a], a, b) == a) return true;
    }
}

// n vertices, m edges of H (at most kMaxCross of each); edge(j) gives edge j's
// two vertices.  Writes C.isbr[j] = 1 for the bridges (0 for the others), and
// with `classes` C.hcls[i] = smallest vertex of the class of H's vertex i.
// Returns false (to every lane) when H's core is too large.
template <class Edge>
__device__ bool solve_contracted(SolveLds& L, const Contract& C, uint32_t n, uint32_t m, bool classes, Edge edge) {
    const uint32_t tid = threadIdx.x;
    uint32_t* par = L.h.par;
    if (tid == 0) { L.nnon = L.ncore = L.nct = L.ncn = L.nuni = 0; }
    for (uint32_t i = tid; i < n; i += kSolveT) par[i] = i;
    for (uint32_t i = tid; i < kMaxCross / 32; i += kSolveT) { L.tree[i] = 0; L.gone[i] = 0; }
    for (uint32_t j = tid; j < m; j += kSolveT) {
        const uint2 ab = edge(j);
        L.h.e[j] = ab.x | ab.y << 16;
    }
    __syncthreads();
    for (uint32_t j = tid; j < m; j += kSolveT) {
        const uint32_t w = L.h.e[j];
        if (h_unite(par, w & 0xffffu, w >> 16)) atomicOr(&L.tree[j >> 5], 1u << (j & 31));
        else atomicAdd(&L.nnon, 1u);
    }
    __syncthreads();
    if (L.nnon == 0) {                       // H is a forest
        for (uint32_t j = tid; j < m; j += kSolveT) C.isbr[j] = 1;
        if (classes)
            for (uint32_t i = tid; i < n; i += kSolveT) C.hcls[i] = C.hroot[i];
        __syncthreads();
        return true;
    }
    // strip the hanging trees: a vertex with one edge left names it by the xor
    for (uint32_t i = tid; i < n; i += kSolveT) par[i] = 0;
    __syncthreads();
    for (uint32_t j = tid; j < m; j += kSolveT) {
        const uint32_t w = L.h.e[j];
        for (uint32_t v : {w & 0xffffu, w >> 16}) {
            atomicAdd(&par[v], 1u << 16);
            atomicXor(&par[v], j);
        }
    }
    for (int round = 0; round < kPeelRounds; round++) {
        __syncthreads();
        if (tid == 0) L.more = 0;
        // the leaves of this round first, then their edges: stripping an edge
        // changes the words of both its ends
        uint32_t last[kMaxCross / kSolveT];
#pragma unroll
        for (int k = 0; k < kMaxCross / kSolveT; k++) {
            const uint32_t v = tid + k * kSolveT;
            const uint32_t w = v < n ? par[v] : 0u;
            last[k] = w >> 16 == 1 ? w & 0xffffu : 0xffffffffu;
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < kMaxCross / kSolveT; k++) {
            const uint32_t j = last[k];
            if (j == 0xffffffffu) continue;
            // both ends of a lone edge may be leaves: the first to mark it acts
            if (atomicOr(&L.gone[j >> 5], 1u << (j & 31)) >> (j & 31) & 1u) continue;
            const uint32_t w = L.h.e[j];
            for (uint32_t x : {w & 0xffffu, w >> 16}) {
                atomicSub(&par[x], 1u << 16);
                atomicXor(&par[x], j);
            }
            L.more = 1;
        }
        __syncthreads();
        if (!L.more) break;
    }
    __syncthreads();
    // the core: vertices with edges left, renumbered
    for (uint32_t i = tid; i < n; i += kSolveT) par[i] = par[i] >> 16 ? atomicAdd(&L.ncore, 1u) : 0xffffffffu;
    __syncthreads();
    const uint32_t nc = L.ncore;
    if (nc > (uint32_t)kCoreV) return false;
    for (uint32_t j = tid; j < m; j += kSolveT) {
        const bool gone = L.gone[j >> 5] >> (j & 31) & 1u;
        C.isbr[j] = gone ? 1u : 0u;
        if (!gone) {
            const uint32_t w = L.h.e[j], c = atomicAdd(&L.nct, 1u);
            C.core[c] = par[w & 0xffffu] | par[w >> 16] << 16;
            C.corej[c] = j;
        }
    }
    __syncthreads();
    const uint32_t mc = L.nct;
    __syncthreads();
    if (tid == 0) L.nct = 0;
    for (uint32_t i = tid; i < nc; i += kSolveT) par[i] = i;
    __syncthreads();
    for (uint32_t c = tid; c < mc; c += kSolveT) {
        const uint32_t w = C.core[c];
        if (h_unite(par, w & 0xffffu, w >> 16)) {
            const uint32_t t = atomicAdd(&L.nct, 1u);
            C.tree[t] = w;
            C.treej[t] = C.corej[c];
        } else {
            C.non[atomicAdd(&L.ncn, 1u)] = w;
        }
    }
    __syncthreads();
    for (uint32_t i = tid; i < nc; i += kSolveT) C.root[i] = par[i] == i;
    __syncthreads();
    const uint32_t n1 = L.nct, n2 = L.ncn;
    for (uint32_t t = tid; t < n1; t += kSolveT) L.small.e1[t] = C.tree[t];
    __syncthreads();
    small_bridges<kCoreV, kSolveT>(
        L.small, nc, n1, n2, [&](uint32_t v) { return C.root[v] != 0; },
        [&](uint32_t k) { return make_uint2(C.non[k] & 0xffffu, C.non[k] >> 16); });
    const uint32_t nk = L.small.nkeys;
    for (uint32_t i = tid; i < nk; i += kSolveT) C.isbr[C.treej[L.small.cur[i]]] = 1;
    __syncthreads();
    if (!classes) return true;
    // classes: H without its bridges, each labelled by its smallest vertex
    uint32_t* low = L.h.e;
    for (uint32_t i = tid; i < n; i += kSolveT) { par[i] = i; low[i] = 0xffffffffu; }
    __syncthreads();
    for (uint32_t j = tid; j < m; j += kSolveT) {
        if (C.isbr[j]) continue;
        const uint2 ab = edge(j);
        if (h_unite(par, ab.x, ab.y)) atomicAdd(&L.nuni, 1u);
    }
    __syncthreads();
    for (uint32_t i = tid; i < n; i += kSolveT) atomicMin(&low[h_find(par, i)], C.hroot[i]);
    __syncthreads();
    for (uint32_t i = tid; i < n; i += kSolveT) C.hcls[i] = low[h_find(par, i)];
    __syncthreads();
    return true;
}

// The answer for the host: bridges (mode 0), classes (1) or classes and bridge
// tree (2).  out: 64 status words -- [1] bridges or classes, [2], [3] |F|, |F'|,
// [4] error word, [5] bridges (the tree's edges), [6] 1 if solved -- and (modes
// 0 and 2) the keys min << 32 | max.
__device__ __forceinline__ void report_contracted(SolveLds& L, const int2* f1, uint32_t c1, uint32_t c2, uint32_t err,
                                                  uint32_t V, const Contract& C, uint32_t m, bool ok, int32_t mode,
                                                  uint32_t* out, uint64_t* keys) {
    if (threadIdx.x == 0) L.nout = 0;
    __syncthreads();
    if (ok)
        for (uint32_t j = threadIdx.x; j < m; j += kSolveT) {
            if (!C.isbr[j]) continue;
            uint32_t a, b;
            if (mode == 0) {
                const int2 e = f1[C.hk[j]];
                a = (uint32_t)e.x;
                b = (uint32_t)e.y;
            } else {
                const uint2 r = C.he[j];
                a = C.hcls[C.hid[r.x] - 1];
                b = C.hcls[C.hid[r.y] - 1];
            }
            const uint32_t p = atomicAdd(&L.nout, 1u);
            if (mode != 1) keys[p] = (uint64_t)min(a, b) << 32 | max(a, b);
        }
    __syncthreads();
    if (threadIdx.x == 0) {
        out[1] = mode == 0 ? L.nout : V - c2 - (ok ? L.nuni : 0u);
        out[2] = c1;
        out[3] = c2;
        out[4] = err;
        out[5] = L.nout;
        out[6] = ok ? 1u : 0u;
        out[8] = 0;
    }
}

}  // namespace br
