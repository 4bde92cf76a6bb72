// The union-find of Algorithm 2 in a workgroup's LDS (included by .hip sources
// only): one 32-bit word per vertex, low half = x - parent in F, high half =
// x - parent in F' (0 = root; V <= 65,536 keeps both in 16 bits).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "device_util.hpp"

namespace br {

typedef uint16_t __attribute__((may_alias)) lds_half;

template <int F>
__device__ __forceinline__ uint32_t half(uint32_t w) { return F ? (w >> 16) : (w & 0xffffu); }

template <int F>
__device__ __forceinline__ uint32_t with_half(uint32_t w, uint32_t h) {
    return F ? ((w & 0xffffu) | (h << 16)) : ((w & 0xffff0000u) | h);
}

// Representative of x, halving the path: reads and stores of one half, so the
// other half, which may be changing under a concurrent hook, is left alone.
// One workgroup's searches are bound by instructions, not by LDS latency (its
// 16 wavefronts share one CU's issue), so the plain loop wins: climbing both
// chains at once or in Rem's order, which needs fewer steps, measured 182 and
// 193 us against 118 for 49,000 edges over 12,345 vertices.
template <int F>
__device__ __forceinline__ uint32_t lfind(uint32_t* q, uint32_t x) {
    lds_half* h = reinterpret_cast<lds_half*>(q) + F;
    uint32_t d = h[2 * x];
    while (d != 0) {
        const uint32_t p = x - d;
        const uint32_t dp = h[2 * p];
        if (dp == 0) return p;
        h[2 * x] = (uint16_t)(d + dp);
        x = p - dp;
        d = h[2 * x];
    }
    return x;
}

template <int F>
__device__ __forceinline__ bool lunite(uint32_t* q, uint32_t u, uint32_t v) {
    for (;;) {
        u = lfind<F>(q, u);
        v = lfind<F>(q, v);
        if (u == v) return false;
        if (u < v) { const uint32_t t = u; u = v; v = t; }
        uint32_t w = q[u];
        for (;;) {
            if (half<F>(w) != 0) break;                       // u was hooked meanwhile
            const uint32_t nw = with_half<F>(w, u - v);
            const uint32_t old = atomicCAS(&q[u], w, nw);
            if (old == w) return true;
            w = old;                                          // other half changed, or u hooked
        }
        u = u - half<F>(w);
    }
}

// Offer (u,v) to F, then to F'.  Both parents come from one 32-bit word per
// endpoint; F' only joins what F joins, so a shared parent in F' rejects the
// edge in both (the usual case once the state is compressed).
__device__ __forceinline__ void loffer(uint32_t* q, uint32_t u, uint32_t v, bool& a1, bool& a2) {
    const uint32_t wu = q[u], wv = q[v];
    const uint32_t p2u = u - (wu >> 16), p2v = v - (wv >> 16);
    a1 = a2 = false;
    if (p2u == p2v) return;
    const uint32_t p1u = u - (wu & 0xffffu), p1v = v - (wv & 0xffffu);
    a1 = p1u != p1v && lunite<0>(q, p1u, p1v);
    if (!a1) a2 = lunite<1>(q, p2u, p2v);
}

// Full path compression of the LDS state (no concurrent hooks: called between
// barriers), so that later edges inside a component hit the shared-parent test.
__device__ void lcompress(uint32_t* q, uint32_t V) {
    for (uint32_t x = threadIdx.x; x < V; x += blockDim.x) {
        const uint32_t w = q[x];
        uint32_t r1 = x - (w & 0xffffu), r2 = x - (w >> 16);
        for (uint32_t d = q[r1] & 0xffffu; d; d = q[r1] & 0xffffu) r1 -= d;
        for (uint32_t d = q[r2] >> 16; d; d = q[r2] >> 16) r2 -= d;
        const uint32_t nw = (x - r1) | ((x - r2) << 16);
        if (nw != w) atomicCAS(&q[x], w, nw);
    }
}


// wavefront-aggregated reservation of slots for F's and F''s accepted edges
// on the packed LDS counter: one atomic and one broadcast per wavefront step
// for both forests (the two were each an LDS atomic plus a permute)
__device__ __forceinline__ void reserve2(uint32_t* ctr, bool a1, bool a2, uint32_t& p1, uint32_t& p2) {
    const uint64_t m1 = __ballot(a1), m2 = __ballot(a2);
    p1 = p2 = 0;
    if ((m1 | m2) == 0) return;
    const int leader = __ffsll((unsigned long long)(m1 | m2)) - 1;
    uint32_t base = 0;
    if (__lane_id() == leader) base = atomicAdd(ctr, (uint32_t)__popcll(m1) | ((uint32_t)__popcll(m2) << 16));
    base = __shfl(base, leader);
    p1 = (base & 0xffffu) + lane_rank(m1);
    p2 = (base >> 16) + lane_rank(m2);
}

}  // namespace br
