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

// representative of x in forest F (path halving on the way)
template <int F>
__device__ __forceinline__ uint32_t uf_find(uint32_t* q, int64_t qs, uint32_t x) {
    uint32_t d = ld(q + qs * (int64_t)x + F);
    while (d != 0) {
        const uint32_t p = x - d;
        const uint32_t dp = ld(q + qs * (int64_t)p + F);
        if (dp == 0) return p;
        st(q + qs * (int64_t)x + F, d + dp);   // x now points at its grandparent
        x = p - dp;
        d = ld(q + qs * (int64_t)x + F);
    }
    return x;
}

// true iff this call merged the components of u and v in forest F
//
// A root that many lanes want to hook is one address, and compare-and-swaps on
// one address queue at the memory side whether they win or fail.  By the time
// v's root is found, u has often been hooked by another lane; a device-scope
// load (past this XCD's caches, which may show a root long hooked) sees that
// without joining the queue.  Measured on 1.5 M random edges over 10^6
// vertices, F and F': 1,400-1,800 us without the load, 215 us with it; 133,072
// over 66,536: 300-800 and 77 us.
template <int F>
__device__ __forceinline__ bool uf_unite(uint32_t* q, int64_t qs, uint32_t u, uint32_t v) {
    for (;;) {
        u = uf_find<F>(q, qs, u);
        v = uf_find<F>(q, qs, v);
        if (u == v) return false;
        if (u < v) { const uint32_t t = u; u = v; v = t; }
        uint32_t* w = q + qs * (int64_t)u + F;
        uint32_t d = __hip_atomic_load(w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (d == 0 && __hip_atomic_compare_exchange_strong(w, &d, u - v, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                           __HIP_MEMORY_SCOPE_AGENT))
            return true;
        u = u - d;   // u was hooked meanwhile: continue from its parent
    }
}

// Offer edge (u,v) to F, then (if rejected) to F'.  su, sv are the
// endpoints' parent words (F low, F' high), loaded earlier with one 8-byte
// load each: however stale, each names an ancestor (or the vertex itself), a
// valid place to start the finds from.
__device__ __forceinline__ void offer_from(uint32_t* q, int64_t qs, uint32_t u, uint32_t v, uint64_t su, uint64_t sv,
                                           bool& a1, bool& a2) {
    const uint32_t p1u = u - (uint32_t)su, p1v = v - (uint32_t)sv;
    a1 = (p1u != p1v) && uf_unite<0>(q, qs, p1u, p1v);
    a2 = false;
    if (!a1) {
        const uint32_t p2u = u - (uint32_t)(su >> 32), p2v = v - (uint32_t)(sv >> 32);
        a2 = (p2u != p2v) && uf_unite<1>(q, qs, p2u, p2v);
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
