// Final step of the batched path on the device for the graphs the persistent
// kernel could not finish itself (the contracted certificate keeps a core of
// cycles): the bridges of each one's certificate, one workgroup per graph,
// entirely in LDS.
//
// The certificate is the one the persistent batched kernel leaves in node 0's
// region of each graph (F from the front, F' from the back, graph-local ids),
// with the roots of F's trees flagged in rootw.

#include <hip/hip_runtime.h>

#include "internal.hpp"
#include "small_bridges.hpp"

namespace br {

namespace {

constexpr int kLimitV = 4096;                 // vertices per small graph (the batched kernel's LDS limit)
constexpr int kSplitV = 1024;                 // graphs up to this size run in smaller workgroups, several per CU

template <int kMaxV, int kST>
__global__ void __launch_bounds__(kST) k_small_bridges(const BatchDev B, const int32_t* list, const uint32_t* nlist,
                                                       uint32_t* out_hdr, uint32_t* out_keys) {
    extern __shared__ __align__(16) unsigned char lds_raw[];
    SmallLds<kMaxV, kST>& L = *reinterpret_cast<SmallLds<kMaxV, kST>*>(lds_raw);
    const int tid = threadIdx.x;
    const int64_t left = *nlist;
    for (int64_t it = blockIdx.x; it < left; it += gridDim.x) {
        const int64_t g = list[it];
        const uint32_t V = (uint32_t)B.V[g];
        const int64_t off = B.noff[g], cap = B.ncap[g], vb = B.vbase[g];
        const uint32_t c1 = min((int64_t)B.ncnt[2 * g], cap);
        const uint32_t n1 = c1, n2 = (uint32_t)min((int64_t)B.ncnt[2 * g + 1], cap - (int64_t)c1);
        if (tid == 0) L.bad = 0;
        __syncthreads();
        const bool ok = V >= 1 && V <= (uint32_t)kMaxV && n1 <= V - 1;
        if (!ok) {
            if (tid == 0) { atomicOr(B.err, 4u); out_hdr[16 + 2 * g] = 0; out_hdr[16 + 2 * g + 1] = 0; }
            __syncthreads();
            continue;
        }
        // ---- F
        for (uint32_t k = tid; k < n1; k += kST) {
            const int2 e = B.cert[off + k];
            if ((uint32_t)e.x >= V || (uint32_t)e.y >= V || e.x == e.y) L.bad = 1;
            L.e1[k] = ((uint32_t)e.x & 0xffffu) | ((uint32_t)e.y << 16);
        }
        __syncthreads();
        if (L.bad) {
            if (tid == 0) { atomicOr(B.err, 4u); out_hdr[16 + 2 * g] = 0; out_hdr[16 + 2 * g + 1] = 0; }
            __syncthreads();
            continue;
        }
        small_bridges<kMaxV, kST>(
            L, V, n1, n2, [&](uint32_t v) { return B.rootw[vb + v] == 0; },
            [&](uint32_t k) {
                const int2 e = B.cert[off + cap - n2 + k];
                return make_uint2((uint32_t)e.x, (uint32_t)e.y);
            });
        // ---- keys
        const uint32_t nk = min(L.nkeys, (uint32_t)kMaxV);
        for (uint32_t i = tid; i < nk; i += kST) {
            const uint32_t e = L.e1[L.cur[i]], a = e & 0xffffu, b = e >> 16;
            L.cur[i] = (min(a, b) << 16) | max(a, b);
        }
        // ---- canonical order (bitonic sort) and output
        uint32_t P = 1;
        while (P < nk) P <<= 1;
        for (uint32_t k = nk + tid; k < P; k += kST) L.cur[k] = 0xffffffffu;
        __syncthreads();
        for (uint32_t k = 2; k <= P; k <<= 1) {
            for (uint32_t j = k >> 1; j > 0; j >>= 1) {
                for (uint32_t i = tid; i < P; i += kST) {
                    const uint32_t q = i ^ j;
                    if (q > i) {
                        const uint32_t x = L.cur[i], y = L.cur[q];
                        if (((i & k) == 0) == (x > y)) { L.cur[i] = y; L.cur[q] = x; }
                    }
                }
                __syncthreads();
            }
        }
        if (tid == 0) {
            L.base = nk ? atomicAdd(out_hdr, nk) : 0u;
            out_hdr[16 + 2 * g] = L.base;
            out_hdr[16 + 2 * g + 1] = nk;
        }
        __syncthreads();
        for (uint32_t k = tid; k < nk; k += kST) out_keys[L.base + k] = L.cur[k];
        __syncthreads();
    }
}

}  // namespace

int32_t small_bridges_max_v() { return kLimitV; }
int32_t small_bridges_split_v() { return kSplitV; }

void launch_small_bridges(const BatchDev& B, int32_t na, int32_t nb, int cus, hipStream_t s, hipStream_t s_b) {
    if (nb > 0)
        hipLaunchKernelGGL((k_small_bridges<kLimitV, 1024>), dim3((unsigned)std::min(nb, cus)), dim3(1024),
                           sizeof(SmallLds<kLimitV, 1024>), s_b, B, (const int32_t*)B.list_b, B.out_hdr + 3, B.out_hdr, B.out_keys);
    if (na > 0)
        hipLaunchKernelGGL((k_small_bridges<kSplitV, 256>), dim3((unsigned)std::min(na, 4 * cus)), dim3(256),
                           sizeof(SmallLds<kSplitV, 256>), s, B, (const int32_t*)B.list_a, B.out_hdr + 2, B.out_hdr, B.out_keys);
}

int prepare_small_bridges() {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_small_bridges<kLimitV, 1024>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)sizeof(SmallLds<kLimitV, 1024>));
    if (e == hipSuccess)
        e = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_small_bridges<kSplitV, 256>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)sizeof(SmallLds<kSplitV, 256>));
    return e == hipSuccess ? 0 : -1;
}

}  // namespace br
