// The lock-free union-find of Algorithm 2 over a state in device memory,
// shared by the kernel files that offer edges to it (included by .hip sources
// only).  For every vertex x and forest f (0 = F, 1 = F') the word q[qs*x + f]
// holds x - parent(x), 0 at a root; cert_kernels.hip has the argument for its
// correctness under concurrent updates.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "device_util.hpp"

namespace br {

__device__ __forceinline__ uint32_t ld(const uint32_t* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
}
__device__ __forceinline__ void st(uint32_t* p, uint32_t v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
}
__device__ __forceinline__ uint64_t ld2(const uint32_t* p) {
    return __hip_atomic_load(reinterpret_cast<const uint64_t*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
}

constexpr int kFreeSteps = 16;   // steps of a search before it begins to shorten the chain
// Steps after which a search stops and its wavefront walks for it.  A walk costs
// up to 2 us per 256 ids, so it has to be rare: with 512 steps the articulation
// points of a mesh row by row (3V edges, V = 10^6) took 2.6 ms, with 2,048 2.0 (as
// without walks); a ring of 20,000 vertices 0.55 and 0.83 ms (5.5 without).
constexpr int kDeepSteps = 2048;

// Unite u and v, whose parents were seen as pu and pv (however stale, each
// names an ancestor or the vertex itself); true iff this call merged their
// components, else pu == pv if they are one component already.  The end whose
// parent is larger moves up, so the search stops where the two chains meet (Rem's
// order; no need to reach the roots), and a root that is reached hooks under the
// other end's parent.  Long searches halve the chain as they go; short ones leave
// no dirty lines behind, which hooks (swaps at the memory side) would have to
// write back first.  A search that is not over after kSteps steps stops where it
// stands (false, pu != pv).
//
// A root that many lanes want to hook is one address, and compare-and-swaps on
// one address queue at the memory side whether they win or fail.  By the time
// the search is over, u has often been hooked by another lane; a device-scope
// load (past this XCD's caches, which may show a root long hooked) sees that
// without joining the queue.  Of a wavefront's lanes at one root the
// first goes ahead and the others go on from what it found (a star whose hub has
// the largest id, 10^6 leaves: 2,300 to 2,800 us with a swap per lane, 129 so).
//
// Measured, F and F': 1.5 M random edges over 10^6 vertices 1,400-1,800 us with
// two full searches and no load before the swap, 215 with the load, 200 in
// Rem's order; 133,072 over 66,536 vertices 300-800, 77, 62 us; 534,288 over
// 267,144 vertices (load) 153, 133 us.
template <int kSteps = kDeepSteps>
__device__ __forceinline__ bool uf_search(uint32_t* q, int64_t qs, uint32_t& u, uint32_t& pu, uint32_t& v, uint32_t& pv) {
    for (int n = 0; pu != pv && n < kSteps; n++) {
        if (pu < pv) {
            uint32_t t = u;
            u = v;
            v = t;
            t = pu;
            pu = pv;
            pv = t;
        }
        if (u == pu) {
            uint32_t* w = q + qs * (int64_t)u;
            uint32_t d = __hip_atomic_load(w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (d == 0) {
                const bool goes = u != (uint32_t)__builtin_amdgcn_readfirstlane((int)u) || lane_rank(__ballot(1)) == 0;
                bool won = false;
                if (goes) {
                    won = __hip_atomic_compare_exchange_strong(w, &d, u - pv, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                               __HIP_MEMORY_SCOPE_AGENT);
                    if (won) d = u - pv;
                }
                const uint32_t first = (uint32_t)__builtin_amdgcn_readfirstlane((int)d);
                if (!goes) d = first;
                if (won) return true;
            }
            pu = u - d;   // u was hooked meanwhile
            continue;
        }
        const uint32_t g = pu - ld(q + qs * (int64_t)pu);
        if (n >= kFreeSteps && g != pu) st(q + qs * (int64_t)u, u - g);
        u = pu;
        pu = g;
    }
    return false;
}

// Root of x (the same in every lane of the wavefront, all of them active), or
// what a stale word shows as one.  The lanes read the words of the 256 ids down
// from x and jump among them, which is where a chain of near ids leads, so a
// walk takes at most one round of about 2 us per 256 ids between x and its
// root, however long the chain.  What it has seen it leaves shortened.
__device__ __forceinline__ uint32_t uf_walk(uint32_t* q, int64_t qs, uint32_t x) {
    constexpr int kW = 4;
    const uint32_t lane = __lane_id();
    for (;;) {
        uint32_t at[kW];                       // offset below x that lane's id leads to
        for (int k = 0; k < kW; k++) {
            const uint32_t o = k * 64 + lane;
            at[k] = o + (o <= x ? ld(q + qs * (int64_t)(x - o)) : 0u);
        }
        uint32_t p = 0;
        bool root = false;
        for (int k = 0; k < kW; k++) {
            const uint32_t lo = k * 64, first = at[k];
            // (a root leads to itself)
            for (int r = 0; r < 6; r++) {
                const uint32_t t = __shfl(at[k], (int)((at[k] - lo) & 63u));
                if (at[k] < lo + 64) at[k] = t;
            }
            const uint32_t o = lo + lane;
            if (at[k] != first) st(q + qs * (int64_t)(x - o), at[k] - o);
            if (p < lo + 64) {                 // the chain comes by this window (uniform)
                const uint32_t t = __shfl(at[k], (int)(p - lo));
                root = t < lo + 64;
                p = t;
                if (root) break;
            }
        }
        x -= p;
        if (root) return x;
    }
}

// x's word in one union-find (words w[qs * x]) set to its root, which is
// returned; called by one thread per vertex, with no hooks meanwhile.  Past
// kFreeSteps plain steps a thread leaves each step it makes where all XCDs see
// it and reads what the others left, so that a long chain takes its logarithm in
// steps.  (Plain loads throughout, every 16th step left behind: the caches show
// the old words, 385 us for a path of 4,000 vertices, 4.2 ms for 10^6.)
__device__ __forceinline__ uint32_t uf_compress(uint32_t* w, int64_t qs, uint32_t x) {
    const uint32_t d = w[qs * (int64_t)x];
    if (d == 0) return x;
    uint32_t r = x - d;
    for (int n = 0; n < kFreeSteps; n++) {
        const uint32_t e = w[qs * (int64_t)r];
        if (e == 0) {
            if (n) w[qs * (int64_t)x] = x - r;
            return r;
        }
        r -= e;
    }
    for (;;) {
        __hip_atomic_store(w + qs * (int64_t)x, x - r, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const uint32_t e = __hip_atomic_load(w + qs * (int64_t)r, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (e == 0) return r;
        r -= e;
    }
}

// For the lanes in m, which hold searches that stand open (in forest `forest` each,
// q its first word; every lane of the wavefront calls it): the first of them gets
// its two roots from a walk of the whole wavefront, and what that leaves shortened
// serves the others.  One lane alone took 270 ns per vertex of a list in vertex
// order: a ring of 200,000 vertices closed after 54 ms, with the walk after 2.4.
__device__ __forceinline__ void uf_help(uint64_t m, uint32_t* q, int64_t qs, int forest, uint32_t& u, uint32_t& pu,
                                        uint32_t& v, uint32_t& pv) {
    const int lane = __ffsll((unsigned long long)m) - 1;
    uint32_t* w = q + __shfl(forest, lane);
#pragma unroll 1
    for (int end = 0; end < 2; end++) {
        const uint32_t r = uf_walk(w, qs, (uint32_t)__shfl((int)(end ? v : u), lane));
        if ((int)__lane_id() == lane) {
            if (end) v = pv = r;
            else u = pu = r;
        }
    }
}

// The wavefront's lanes (all of them, active or not) unite their pairs in one
// union-find.
__device__ __forceinline__ bool uf_unite(uint32_t* q, int64_t qs, bool active, uint32_t u, uint32_t pu, uint32_t v, uint32_t pv) {
    bool merged = false;
    for (bool open = active;;) {
        if (open) {
            merged = uf_search(q, qs, u, pu, v, pv);
            open = !merged && pu != pv;
        }
        const uint64_t m = __ballot(open);
        if (!m) return merged;
        uf_help(m, q, qs, 0, u, pu, v, pv);
    }
}

// Root of x, halving the chain on the way
__device__ __forceinline__ uint32_t uf_find(uint32_t* q, int64_t qs, uint32_t x) {
    uint32_t d = ld(q + qs * (int64_t)x);
    while (d != 0) {
        const uint32_t p = x - d, dp = ld(q + qs * (int64_t)p);
        if (dp == 0) return p;
        st(q + qs * (int64_t)x, d + dp);
        x = p - dp;
        d = ld(q + qs * (int64_t)x);
    }
    return x;
}

// Unite u and v, lane by lane: kFreeSteps steps in Rem's order, then root under
// root, which keeps the chains of a list in vertex order short.  (For tree edges,
// each of which joins two components.  Classes, 3V edges of a mesh row by row,
// V = 10^6: 1,725 us in k_class_tree in Rem's order, 137 so; a path 26 us so,
// 630 and more root under root alone.)
__device__ __forceinline__ void root_unite(uint32_t* q, int64_t qs, uint32_t u, uint32_t v) {
    uint32_t pu = u - ld(q + qs * (int64_t)u), pv = v - ld(q + qs * (int64_t)v);
    if (uf_search<kFreeSteps>(q, qs, u, pu, v, pv) || pu == pv) return;
    for (;;) {
        u = uf_find(q, qs, u);
        v = uf_find(q, qs, v);
        if (u == v) return;
        if (u < v) {
            const uint32_t t = u;
            u = v;
            v = t;
        }
        uint32_t* w = q + qs * (int64_t)u;
        uint32_t d = __hip_atomic_load(w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (d == 0 && __hip_atomic_compare_exchange_strong(w, &d, u - v, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                           __HIP_MEMORY_SCOPE_AGENT))
            return;
        u -= d;
    }
}

// Offer edge (u,v) (the lanes that are active) to F, then (if rejected) to F'.
// su, sv are the endpoints' parent words (F low, F' high), loaded earlier with
// one 8-byte load each.  F' only joins what F joins, so a shared parent in F'
// rejects the edge in both.  Every lane of the wavefront calls it.
__device__ __forceinline__ void offer_from(uint32_t* q, int64_t qs, bool active, uint32_t u, uint32_t v, uint64_t su,
                                           uint64_t sv, bool& a1, bool& a2) {
    const uint32_t p1u = u - (uint32_t)su, p1v = v - (uint32_t)sv;
    const uint32_t p2u = u - (uint32_t)(su >> 32), p2v = v - (uint32_t)(sv >> 32);
    a1 = a2 = false;
    uint32_t x = u, px = p1u, y = v, py = p1v;
    int forest = 0;
    for (bool open = active && p2u != p2v;;) {
        if (open) {
            if (forest == 0) {
                a1 = uf_search(q, qs, x, px, y, py);
                if (px == py && !a1) {
                    forest = 1;
                    x = u;
                    px = p2u;
                    y = v;
                    py = p2v;
                }
            }
            if (forest == 1) a2 = uf_search(q + 1, qs, x, px, y, py);
            open = !a1 && !a2 && px != py;
        }
        const uint64_t m = __ballot(open);
        if (!m) return;
        uf_help(m, q, qs, forest, x, px, y, py);
    }
}

// Accepted edges of one workgroup tile are staged in LDS (F from the front,
// F' from the back of the stage), then the tile reserves its ranges in the
// node's region with one global atomic per forest and copies them out.  Every
// lane of the workgroup must call these (ballots and barriers).
template <int kTile>
struct StageT {
    int2 e[kTile];
    uint32_t n1, n2;
    uint32_t base1, base2;
};

template <int kTile>
__device__ __forceinline__ void stage_reset(StageT<kTile>& S) {
    if (threadIdx.x == 0) { S.n1 = 0; S.n2 = 0; }
    __syncthreads();
}

template <int kTile>
__device__ __forceinline__ void stage_put(StageT<kTile>& S, bool a1, bool a2, int2 e) {
    const uint64_t m1 = __ballot(a1), m2 = __ballot(a2);
    const int lane = __lane_id();
    if (m1) {
        const int leader = __ffsll((unsigned long long)m1) - 1;
        uint32_t base = 0;
        if (lane == leader) base = atomicAdd(&S.n1, (uint32_t)__popcll(m1));
        base = __shfl(base, leader);
        if (a1) S.e[base + lane_rank(m1)] = e;
    }
    if (m2) {
        const int leader = __ffsll((unsigned long long)m2) - 1;
        uint32_t base = 0;
        if (lane == leader) base = atomicAdd(&S.n2, (uint32_t)__popcll(m2));
        base = __shfl(base, leader);
        if (a2) S.e[kTile - 1 - (base + lane_rank(m2))] = e;
    }
}

// cnt[0], cnt[1]: the region's counters; its pairs are region[0, cap)
template <int kTile>
__device__ __forceinline__ void stage_flush(StageT<kTile>& S, uint32_t* cnt, int2* region, int64_t cap, uint32_t* err) {
    __syncthreads();
    const uint32_t n1 = S.n1, n2 = S.n2;
    if (threadIdx.x == 0) {
        S.base1 = n1 ? atomicAdd(cnt, n1) : 0;
        S.base2 = n2 ? atomicAdd(cnt + 1, n2) : 0;
    }
    __syncthreads();
    const int64_t b1 = S.base1, b2 = S.base2;
    for (uint32_t k = threadIdx.x; k < n1 + n2; k += blockDim.x) {
        int64_t pos;
        int2 e;
        if (k < n1) { pos = b1 + k; e = S.e[k]; }
        else { pos = b2 + (k - n1); e = S.e[kTile - 1 - (k - n1)]; }
        if (pos >= cap) { atomicOr(err, 2u); continue; }
        region[k < n1 ? pos : cap - 1 - pos] = e;
    }
}

}  // namespace br
