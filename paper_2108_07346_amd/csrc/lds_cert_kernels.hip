// The certificate of a graph of up to 8,192 vertices with the union-find in
// one workgroup's LDS (16-bit offsets of both forests in one word per vertex),
// and for short lists the final step in the same launch.
//
// What bounds it: a search step in LDS takes about 0.1 us against 1 us and more
// through the caches, so one workgroup with its state in LDS is faster than
// hundreds that share one in memory as long as it has few edges to offer.
// Short lists (P.lds_whole) are offered whole.  Of longer ones it takes rows
// spread over the list, 2V or 3V edges, after which F' is nearly complete; its
// state, compressed, then goes to memory together with the table of F'
// components (16-bit codes: the root's id + 1), and k_filter sends the rest of
// the list past the table on every CU (fused_kernels.hip).
#include <hip/hip_runtime.h>

#include "contract.hpp"
#include "device_util.hpp"
#include "internal.hpp"
#include "lds_union_find.hpp"

namespace br {

namespace {

constexpr int kT = kSolveT;
constexpr int kU = 4;                       // edges per thread and step

struct LdsHead {
    uint32_t n12, base, ncross, nvert;      // F / F' counts packed in the first
};

__global__ void __launch_bounds__(kT) k_lds_cert(DevBufs B, int64_t E, int32_t Vi, int64_t cap, int32_t mul, int32_t whole,
                                                 int64_t* off_out, int64_t* cap_out, uint32_t* code, Contract C,
                                                 int32_t mode, uint32_t* out, uint64_t* keys, int32_t* label) {
    extern __shared__ __align__(16) unsigned char raw[];
    __shared__ LdsHead H;
    uint32_t* q = reinterpret_cast<uint32_t*>(raw);
    const uint32_t V = (uint32_t)Vi, tid = threadIdx.x;
    for (uint32_t x = tid; x < V; x += kT) q[x] = 0;
    if (C.hid)
        for (uint32_t x = tid; x < V + kContractCounters; x += kT) C.hid[x] = 0;
    if (tid == 0) {
        H.n12 = H.ncross = H.nvert = 0;
        *B.err = 0;
        off_out[0] = 0;
        cap_out[0] = cap;
    }
    __syncthreads();
    // ---- edges
    const int64_t nrows = (E + kRow - 1) / kRow, nsel = (nrows + mul - 1) / mul;
    constexpr int64_t kStepRows = kT / kRow * kU;
    auto load = [&](int64_t sel0, int2 (&e)[kU]) {
#pragma unroll
        for (int j = 0; j < kU; j++) {
            const int64_t sel = sel0 + j * (kT / kRow) + tid / kRow;
            const int64_t i = sel * mul * kRow + tid % kRow;
            e[j] = make_int2(-1, -2);                                  // past the end
            if (sel < nsel && i < E) {
                e[j] = i < B.split ? B.edges[i] : B.edges2[i - B.split];
                if ((uint32_t)e[j].x >= V || (uint32_t)e[j].y >= V) {
                    atomicOr(B.err, 1u);
                    e[j] = make_int2(-1, -2);
                }
            }
        }
    };
    int2 cur[kU], nxt[kU];
    load(0, cur);
    int64_t next_cmp = 2 * (int64_t)V;
    for (int64_t sel = 0; sel < nsel; sel += kStepRows) {
        if (sel * kRow >= next_cmp) {
            __syncthreads();
            lcompress(q, V);
            __syncthreads();
            next_cmp *= 4;
        }
        load(sel + kStepRows, nxt);
#pragma unroll
        for (int j = 0; j < kU; j++) {
            const int2 e = cur[j];
            bool a1 = false, a2 = false;
            if (e.x >= 0) loffer(q, (uint32_t)e.x, (uint32_t)e.y, a1, a2);
            uint32_t p1, p2;
            reserve2(&H.n12, a1, a2, p1, p2);
            if (a1) { if (p1 < cap) B.cert[p1] = e; else atomicOr(B.err, 2u); }
            if (a2) { if (p2 < cap) B.cert[cap - 1 - p2] = e; else atomicOr(B.err, 2u); }
        }
#pragma unroll
        for (int j = 0; j < kU; j++) cur[j] = nxt[j];
    }
    __syncthreads();
    lcompress(q, V);
    __syncthreads();
    // ---- the state, compressed, for the steps that read it from memory
    for (uint32_t x = tid; x < V; x += kT) {
        const uint32_t w = q[x];
        reinterpret_cast<uint2*>(B.state)[x] = make_uint2(w & 0xffffu, w >> 16);
    }
    if (!whole)
        for (uint32_t x = tid; x < V; x += kT) reinterpret_cast<uint16_t*>(code)[x] = (uint16_t)(x - (q[x] >> 16) + 1);
    const uint32_t n1 = H.n12 & 0xffffu, n2 = H.n12 >> 16;
    if (tid == 0) {
        B.cnt[0] = n1;
        B.cnt[1] = n2;
    }
    if (!whole || mode < 0) return;
    // ---- final step: the edges of F that cross components of F'
    for (uint32_t k = tid; k < n1; k += kT) {
        const int2 e = B.cert[k];
        const uint32_t a = (uint32_t)e.x - (q[e.x] >> 16), b = (uint32_t)e.y - (q[e.y] >> 16);
        if (a == b) continue;
        const uint32_t p = atomicAdd(&H.ncross, 1u);
        if (p >= (uint32_t)kMaxCross) continue;
        C.he[p] = make_uint2(a, b);
        C.hk[p] = k;
        C.hid[a] = 1;
        C.hid[b] = 1;
    }
    __syncthreads();
    for (uint32_t x = tid; x < V; x += kT)
        if (C.hid[x]) {
            const uint32_t i = atomicAdd(&H.nvert, 1u);
            C.hid[x] = i + 1;
            if (i < (uint32_t)kMaxCross) C.hroot[i] = x;
        }
    __syncthreads();
    const uint32_t n = H.nvert, m = H.ncross;
    SolveLds& L = *reinterpret_cast<SolveLds*>(raw);                   // the state is not needed any more
    bool ok = n <= (uint32_t)kMaxCross && m <= (uint32_t)kMaxCross;
    if (ok) ok = solve_contracted(L, C, n, m, mode != 0, [&](uint32_t j) {
            const uint2 r = C.he[j];
            return make_uint2(C.hid[r.x] - 1, C.hid[r.y] - 1);
        });
    __syncthreads();
    report_contracted(L, B.cert, n1, n2, *B.err, V, C, m, ok, mode, out, keys);
    if (ok && mode != 0)
        for (uint32_t x = tid; x < V; x += kT) {
            const uint32_t r = x - B.state[2 * x + 1], h = C.hid[r];
            label[x] = (int32_t)(h ? C.hcls[h - 1] : r);
        }
}

}  // namespace

// Vertices up to which this plan is the faster one: one CU offers an edge in
// 2 to 3 ns, and a graph needs about 2V of them before the table is worth
// anything (512,000 edges, query with this plan / with stages 1 and 2 on all
// CUs: V = 2,000 62 / 93 us, 4,000 77 / 94, 8,000 123 / 121, 16,000 172 / 122).
constexpr int32_t kLdsV = 8192;

// Whether the list is offered whole, and the stride of the rows taken else.
// Whole against rows: V = 1,000 45 / 49 us at 16,000 edges, 64 / 51 at 64,000;
// V = 4,000 82 / 102 at 16,000, 97 / 96 at 32,000; V = 8,000 118 / 129 at
// 32,000, 148 / 123 at 64,000.  Rows of 3V edges leave fewer for the searches
// in memory (V = 1,000, 512,000 edges: 2V 61, 3V 54 us); past 4,096 vertices
// 2V is faster (V = 8,000: 123 and 131 us).
bool plan_lds(Plan& P) {
    const int64_t E = P.E, V = P.V;
    if (V > kLdsV) return false;
    P.lds_whole = E <= std::max<int64_t>(16384, std::min<int64_t>(8 * V, 32768));
    const int64_t sample = (V <= 4096 ? 3 : 2) * V;
    P.s1 = P.s2 = P.lds_whole ? 1 : (int32_t)std::max<int64_t>(2, std::min<int64_t>(E / sample, 1 << 20));
    P.code_per = P.lds_whole ? 0 : 2;
    P.code_words = P.lds_whole ? 0 : (int32_t)(((V + 1) / 2 + 3) & ~int64_t(3));
    return true;
}

int lds_cert_prepare() {
    static OncePerDevice once;
    const hipError_t e = once([] {
        return hipFuncSetAttribute(reinterpret_cast<const void*>(&k_lds_cert), hipFuncAttributeMaxDynamicSharedMemorySize,
                                   160 * 1024 - 256);
    });
    return e == hipSuccess ? BR_OK : hip_fail(e, "hipFuncSetAttribute(k_lds_cert)");
}

int launch_lds_cert(const Plan& P, const DevBufs& B, const FusedBufs& F, const Contract& C, int mode, uint32_t* h_status,
                    void* h_data, uint64_t* h_tree, hipStream_t s) {
    const bool fin = P.lds_whole && mode >= 0;
    const size_t lds = std::max<size_t>(4 * (size_t)P.V, fin ? sizeof(SolveLds) : 0);
    hipLaunchKernelGGL(k_lds_cert, dim3(1), dim3(kT), lds, s, B, P.E, P.V, P.cap[0], P.s2, P.lds_whole ? 1 : 0,
                       const_cast<int64_t*>(B.off), const_cast<int64_t*>(B.cap), F.code, C, fin ? mode : -1, h_status,
                       mode == 0 ? reinterpret_cast<uint64_t*>(h_data) : h_tree, reinterpret_cast<int32_t*>(h_data));
    if (P.lds_whole) return 1;
    launch_filter_rest(P, B, F, s);
    return 2;
}

}  // namespace br
