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

// Unite u and v, whose parents were seen as pu and pv (however stale, each
// names an ancestor or the vertex itself); true iff this call merged their
// components.  The end whose parent is larger moves up, so the search stops
// where the two chains meet (Rem's order; no need to reach the roots), and a
// root that is reached hooks under the other end's parent.  Long searches halve
// the chain as they go; short ones leave no dirty lines behind, which hooks
// (swaps at the memory side) would have to write back first.
//
// A root that many lanes want to hook is one address, and compare-and-swaps on
// one address queue at the memory side whether they win or fail.  By the time
// the search is over, u has often been hooked by another lane; a device-scope
// load (past this XCD's caches, which may show a root long hooked) sees that
// without joining the queue.
//
// Measured, F and F': 1.5 M random edges over 10^6 vertices 1,400-1,800 us with
// two full searches and no load before the swap, 215 with the load, 200 in
// Rem's order; 133,072 over 66,536 vertices 300-800, 77, 62 us; 534,288 over
// 267,144 vertices (load) 153, 133 us.
template <int F>
__device__ __forceinline__ bool uf_unite(uint32_t* q, int64_t qs, uint32_t u, uint32_t pu, uint32_t v, uint32_t pv) {
    for (int n = 0;; n++) {
        if (pu == pv) return false;
        if (pu < pv) {
            uint32_t t = u;
            u = v;
            v = t;
            t = pu;
            pu = pv;
            pv = t;
        }
        if (u == pu) {
            uint32_t* w = q + qs * (int64_t)u + F;
            uint32_t d = __hip_atomic_load(w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (d == 0 && __hip_atomic_compare_exchange_strong(w, &d, u - pv, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                               __HIP_MEMORY_SCOPE_AGENT))
                return true;
            pu = u - d;   // u was hooked meanwhile
            continue;
        }
        const uint32_t g = pu - ld(q + qs * (int64_t)pu + F);
        if (n >= kFreeSteps && g != pu) st(q + qs * (int64_t)u + F, u - g);
        u = pu;
        pu = g;
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

// Offer edge (u,v) to F, then (if rejected) to F'.  su, sv are the endpoints'
// parent words (F low, F' high), loaded earlier with one 8-byte load each.
// F' only joins what F joins, so a shared parent in F' rejects the edge in both.
__device__ __forceinline__ void offer_from(uint32_t* q, int64_t qs, uint32_t u, uint32_t v, uint64_t su, uint64_t sv,
                                           bool& a1, bool& a2) {
    const uint32_t p1u = u - (uint32_t)su, p1v = v - (uint32_t)sv;
    const uint32_t p2u = u - (uint32_t)(su >> 32), p2v = v - (uint32_t)(sv >> 32);
    a1 = a2 = false;
    if (p2u == p2v) return;
    a1 = uf_unite<0>(q, qs, u, p1u, v, p1v);
    if (!a1) a2 = uf_unite<1>(q, qs, u, p2u, v, p2v);
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
