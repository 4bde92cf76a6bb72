// Final step over the contracted certificate (contract.hpp has the reason why
// contracting the components of F' keeps bridges and classes): the edges of F
// that cross components of F' are collected by all workgroups, then one
// workgroup solves what is left, and the answer goes straight to pinned host
// memory.  What bounds it is latency: three launches in a row for bridges, four
// for labels, where the tour-based step over all of F takes eleven and more.
#include <hip/hip_runtime.h>

#include "contract.hpp"
#include "device_util.hpp"
#include "internal.hpp"

namespace br {

namespace {

// Steps up a chain of F' that k_cross takes.  A shuffled list leaves chains of
// a few steps (32 do for every one tried); one in vertex order chains of up to V
// (200,000 vertices on a path, each edge four times: 75 ms in k_cross).  k_cross
// then gives up, and the call compresses the state and takes the step again
// (launch_contract_again).  Each vertex to the next twenty, V = 10^6, one query:
// 2.01 ms with 128 steps, 1.91 with 64, 1.90 with 32.
constexpr int kRootSteps = 64;

// x moved up to its root in F' (no shortcut stores: the state is read by every
// workgroup); false if that is more than kRootSteps away
__device__ __forceinline__ bool root2(const uint32_t* q, int64_t qs, uint32_t& x) {
    for (int n = 0; n < kRootSteps; n++) {
        const uint32_t d = q[qs * (int64_t)x + 1];
        if (d == 0) return true;
        x -= d;
    }
    return false;
}

// Collects the crossing edges of F: the roots of their ends at C.he, their
// place in F at C.hk; every root gets a number in H (C.hid: 1 + number).  One
// reservation per block on each counter; past kMaxCross edges nothing more is
// collected (the tour-based step takes over).
__global__ void __launch_bounds__(kSolveT) k_cross(const int2* f1, const uint32_t* cnt, const uint32_t* q, int64_t qs,
                                                   Contract C) {
    __shared__ uint32_t ne, nv, be, bv;
    const int64_t n1 = cnt[0];
    for (int64_t base = blockIdx.x * (int64_t)kSolveT; base < n1; base += (int64_t)gridDim.x * kSolveT) {
        if (threadIdx.x == 0) { ne = 0; nv = 0; }
        __syncthreads();
        const int64_t k = base + threadIdx.x;
        uint32_t r[2] = {0, 0}, at = 0, id[2] = {0, 0};
        bool cross = false, took[2] = {false, false};
        if (k < n1) {
            const int2 e = f1[k];
            r[0] = (uint32_t)e.x;
            r[1] = (uint32_t)e.y;
            const bool near = root2(q, qs, r[0]) && root2(q, qs, r[1]);
            cross = near && r[0] != r[1];
            if (!near) *C.deep = 1;
        }
        const uint64_t m = __ballot(cross);
        if (m) {
            const int leader = __ffsll((unsigned long long)m) - 1;
            if (__lane_id() == leader) at = atomicAdd(&ne, (uint32_t)__popcll(m));
            at = __shfl(at, leader) + lane_rank(m);
            for (int t = 0; t < 2; t++) {
                // a device-scope look first: many edges share a large component's root
                took[t] = cross && __hip_atomic_load(&C.hid[r[t]], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0 &&
                          atomicCAS(&C.hid[r[t]], 0u, 0xffffffffu) == 0;
                if (took[t]) id[t] = atomicAdd(&nv, 1u);
            }
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            be = ne ? atomicAdd(&C.hcnt[1], ne) : 0;
            bv = nv ? atomicAdd(&C.hcnt[0], nv) : 0;
        }
        __syncthreads();
        if (cross && be + at < (uint32_t)kMaxCross) {
            C.he[be + at] = make_uint2(r[0], r[1]);
            C.hk[be + at] = (uint32_t)k;
        }
        for (int t = 0; t < 2; t++)
            if (took[t]) {
                C.hid[r[t]] = bv + id[t] + 1;
                if (bv + id[t] < (uint32_t)kMaxCross) C.hroot[bv + id[t]] = r[t];
            }
        const bool full = be >= (uint32_t)kMaxCross;
        __syncthreads();
        if (full) break;
    }
}

// one workgroup solves H and reports to host memory
__global__ void __launch_bounds__(kSolveT) k_solve(const int2* f1, const uint32_t* cnt, const uint32_t* err, int32_t V,
                                                   Contract C, int32_t mode, uint32_t* out, uint64_t* keys) {
    extern __shared__ __align__(16) unsigned char raw[];
    SolveLds& L = *reinterpret_cast<SolveLds*>(raw);
    const uint32_t n = C.hcnt[0], m = C.hcnt[1], deep = *C.deep;
    bool ok = !deep && n <= (uint32_t)kMaxCross && m <= (uint32_t)kMaxCross;
    if (ok) ok = solve_contracted(L, C, n, m, mode != 0, [&](uint32_t j) {
            const uint2 r = C.he[j];
            return make_uint2(C.hid[r.x] - 1, C.hid[r.y] - 1);
        });
    __syncthreads();
    report_contracted(L, f1, cnt[0], cnt[1], *err, (uint32_t)V, C, m, ok, mode, out, keys);
    if (threadIdx.x == 0) {
        *C.solved = ok ? 1u : 0u;
        if (deep) out[8] = 1;
    }
}

// class labels of all vertices, straight to host memory (every vertex that is not
// alone is an end of an edge of F, so k_cross has been up its chain)
__global__ void __launch_bounds__(256) k_labels(const uint32_t* q, int64_t qs, int32_t V, Contract C,
                                                const uint32_t* solved, int32_t* label) {
    if (!*solved) return;
    GRID_LOOP(x, (int64_t)V) {
        uint32_t r = (uint32_t)x;
        root2(q, qs, r);
        const uint32_t h = C.hid[r];
        label[x] = (int32_t)(h ? C.hcls[h - 1] : r);
    }
}

}  // namespace

int contract_prepare() {
    static OncePerDevice once;
    const hipError_t e = once([] {
        return hipFuncSetAttribute(reinterpret_cast<const void*>(&k_solve), hipFuncAttributeMaxDynamicSharedMemorySize,
                                   (int)sizeof(SolveLds));
    });
    return e == hipSuccess ? BR_OK : hip_fail(e, "hipFuncSetAttribute(k_solve)");
}

size_t contract_clear_words(int32_t V) { return (size_t)V + 64; }
size_t contract_words() { return 11 * (size_t)kMaxCross; }

Contract contract_carve(uint32_t* cleared, uint32_t* scratch, int32_t V) {
    Contract C;
    C.hid = cleared;
    C.hcnt = cleared + V;
    C.solved = C.hcnt + 2;
    C.deep = C.hcnt + 3;
    uint32_t* p = scratch;
    auto take = [&](size_t k) { uint32_t* r = p; p += k * kMaxCross; return r; };
    C.he = reinterpret_cast<uint2*>(take(2));
    C.hk = take(1);
    C.hroot = take(1);
    C.hcls = take(1);
    C.isbr = take(1);
    C.core = take(1);
    C.corej = take(1);
    C.tree = take(1);
    C.treej = take(1);
    C.non = take(1);
    C.root = C.core;          // the core's edges are read before its roots are written
    return C;
}

void launch_contract(const Plan& P, const DevBufs& B, const Contract& C, int mode, uint32_t* h_status, void* h_data,
                     uint64_t* h_tree, hipStream_t s) {
    const int2* f1 = B.cert + P.off[0];
    const int64_t nf = std::max<int64_t>(1, std::min<int64_t>(P.E, (int64_t)P.V - 1));
    hipLaunchKernelGGL(k_cross, dim3((unsigned)std::min<int64_t>((nf + kSolveT - 1) / kSolveT, 1024)), dim3(kSolveT), 0, s,
                       f1, (const uint32_t*)B.cnt, (const uint32_t*)B.state, B.qs, C);
    hipLaunchKernelGGL(k_solve, dim3(1), dim3(kSolveT), sizeof(SolveLds), s, f1, (const uint32_t*)B.cnt,
                       (const uint32_t*)B.err, P.V, C, mode, h_status,
                       mode == 0 ? reinterpret_cast<uint64_t*>(h_data) : h_tree);
    if (mode != 0)
        hipLaunchKernelGGL(k_labels, dim3(grid_for(P.V)), dim3(256), 0, s, (const uint32_t*)B.state, B.qs, P.V, C,
                           (const uint32_t*)C.solved, reinterpret_cast<int32_t*>(h_data));
}

void launch_contract_again(const Plan& P, const DevBufs& B, const Contract& C, int mode, uint32_t* h_status, void* h_data,
                           uint64_t* h_tree, hipStream_t s) {
    launch_flatten(P, B, s);
    launch_fill_u32(C.hid, (int64_t)contract_clear_words(P.V), 0u, s);
    launch_contract(P, B, C, mode, h_status, h_data, h_tree, s);
}

}  // namespace br
