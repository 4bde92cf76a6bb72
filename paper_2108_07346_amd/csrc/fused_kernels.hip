// The certificate of a whole edge list in one pass (the phase tree of Section
// III with every level folded into its root).
//
// Node (0, q) of the tree is the certificate of its chunks' union, and a
// certificate of that union taken from the edges themselves is as good as one
// taken from two certificates (both keep the same connectivity, Section III).
// Between machines the lower certificates are what travels; on one GPU every
// chunk's edges are at hand, and the lower levels only add work: each chunk
// offers and hooks up to 2(V-1) edges of its own.  So the root's certificate
// is built directly: F and F' (Algorithm 2) over all the edges, by one
// union-find that every workgroup shares.
//
// What bounds it: the edge list is read once (8 bytes per edge), but an edge
// offered to the union-find costs dependent random reads, and the ~2V edges
// that are accepted cost a memory-side swap each.  Three stages keep the
// searches off the long part of the list:
//   1. rows of 512 edges spread over the whole list, about 2V edges: most
//      hooks happen here, one edge per thread;
//   2. (lists over 16V edges) 6V more edges in the same way, after a full
//      path compression: F' becomes nearly complete;
//   3. the rest, against a table in LDS.  An edge of F' joins vertices that F
//      already connects, so the components of F' lie inside those of F, and an
//      edge whose endpoints share a component of F' is rejected by both
//      forests -- now and ever after, since components only grow.  The table
//      holds a code per vertex that names its component of F' as of the end of
//      stage 2 (16, 8, 4, 2 or 1 bits, as many as fit 144 KB; 0 = unnamed:
//      components beyond the codes, taken largest first).  Equal codes reject
//      the edge with two LDS reads; the others go to a list of the wavefront
//      and are offered to the union-find 64 at a time.
#include <hip/hip_runtime.h>

#include "device_util.hpp"
#include "internal.hpp"
#include "union_find.hpp"

namespace br {

namespace {

constexpr int kRowBlock = 512;
constexpr int kMaxRows = 8;            // rows per workgroup of the offering stages
constexpr int kFilterBlock = 1024;
constexpr int kFilterWaves = kFilterBlock / 64;
constexpr int kListCap = 128;          // edges a wavefront's list holds
constexpr int kFilterLds = 160 * 1024;
constexpr int kListBytes = kFilterWaves * kListCap * (int)sizeof(int2);
constexpr int kTabBytes = kFilterLds - kListBytes - 256;     // and the static LDS

// row taken as the sel-th of a stage: the multiples of `mul`, or (div > 0) the
// multiples of `mul` that are not multiples of mul * (div + 1)
__device__ __forceinline__ int64_t stage_row(uint32_t sel, int32_t mul, uint32_t div) {
    return (int64_t)mul * (int64_t)(div ? sel + sel / div + 1u : sel);
}

__device__ __forceinline__ int2 edge_at(const DevBufs& B, int64_t i) {
    return i < B.split ? B.edges[i] : B.edges2[i - B.split];
}

// zeroes [p, p + n16) and writes node 0's region table
__global__ void __launch_bounds__(256) k_fused_init(uint4* p, int64_t n16, int64_t* off, int64_t* cap, int64_t cap0) {
    GRID_LOOP(i, n16) p[i] = make_uint4(0, 0, 0, 0);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        off[0] = 0;
        cap[0] = cap0;
    }
}

// Stages 1 and 2 (and 3 without a table): workgroup b offers rows
// [b * rpw, (b + 1) * rpw) of the stage.
__global__ void __launch_bounds__(kRowBlock) k_rows(DevBufs B, int64_t E, int32_t V, int64_t cap, uint32_t nsel,
                                                    int32_t mul, uint32_t div, int32_t rpw) {
    __shared__ StageT<kRow * kMaxRows> S;
    stage_reset(S);
    const uint32_t s0 = blockIdx.x * (uint32_t)rpw, s1 = min(nsel, s0 + (uint32_t)rpw);
    for (uint32_t sel = s0; sel < s1; sel++) {
        const int64_t i = stage_row(sel, mul, div) * kRow + threadIdx.x;
        bool a1 = false, a2 = false;
        int2 e = make_int2(0, 0);
        uint64_t su = 0, sv = 0;
        bool ok = false;
        if (i < E) {
            e = edge_at(B, i);
            ok = (uint32_t)e.x < (uint32_t)V && (uint32_t)e.y < (uint32_t)V;
            if (ok) {
                su = ld2(B.state + B.qs * (int64_t)e.x);
                sv = ld2(B.state + B.qs * (int64_t)e.y);
            } else {
                atomicOr(B.err, 1u);
            }
        }
        offer_from(B.state, B.qs, ok, (uint32_t)e.x, (uint32_t)e.y, su, sv, a1, a2);
        stage_put(S, a1, a2, e);
    }
    stage_flush(S, B.cnt, B.cert, cap, B.err);
}

// Full path compression of both forests; with rcode, every root of F' takes a
// code (1..65535, in no particular order; 0 once they are used up).
__global__ void __launch_bounds__(256) k_flatten(uint32_t* q, int64_t qs, int32_t V, uint32_t* rcode, uint32_t* ncode) {
    const int64_t n = ((int64_t)V + 63) & ~int64_t(63);        // whole wavefronts, for the ballots
    GRID_LOOP(x, n) {
        bool root = false;
        if (x < V) {
            uf_compress(q, qs, (uint32_t)x);
            root = uf_compress(q + 1, qs, (uint32_t)x) == (uint32_t)x;
        }
        if (!rcode) continue;
        const uint64_t m = __ballot(root);
        if (!m) continue;
        const int leader = __ffsll((unsigned long long)m) - 1;
        uint32_t base = 0;
        if (__lane_id() == leader) base = atomicAdd(ncode, (uint32_t)__popcll(m));
        base = __shfl(base, leader);
        const uint32_t c = base + lane_rank(m) + 1;
        if (root) rcode[x] = c <= 0xffffu ? c : 0u;
    }
}

// The same for one union-find alone (its words q[x]); with names, every root's
// code is written (0 without).
__global__ void __launch_bounds__(256) k_flatten1(uint32_t* q, int32_t V, uint32_t* rcode, uint32_t* ncode, int32_t names) {
    const int64_t n = ((int64_t)V + 63) & ~int64_t(63);
    GRID_LOOP(x, n) {
        const bool root = x < V && uf_compress(q, 1, (uint32_t)x) == (uint32_t)x;
        const uint64_t m = __ballot(root);
        if (!m) continue;
        uint32_t c = 0;
        if (names) {
            const int leader = __ffsll((unsigned long long)m) - 1;
            uint32_t base = 0;
            if (__lane_id() == leader) base = atomicAdd(ncode, (uint32_t)__popcll(m));
            c = __shfl(base, leader) + lane_rank(m) + 1;
            if (c > 0xffffu) c = 0;
        }
        if (root) rcode[x] = c;
    }
}

// Fewer than 16 bits per code: the components that hold most of up to 1,024
// evenly spread vertices take the codes 1..ncodes (one workgroup; the state is
// compressed).
constexpr int kPick = 1024;
__global__ void __launch_bounds__(kPick) k_pick(const uint32_t* q, int64_t qs, int32_t V, int32_t samples,
                                                int32_t ncodes, uint32_t* rcode) {
    __shared__ uint32_t key[2 * kPick], num[2 * kPick];
    __shared__ __align__(16) uint32_t freq[kPick];
    __shared__ uint32_t root[kPick], nd;
    for (int i = threadIdx.x; i < 2 * kPick; i += kPick) { key[i] = 0; num[i] = 0; }
    if (threadIdx.x == 0) nd = 0;
    freq[threadIdx.x] = 0;
    __syncthreads();
    if ((int)threadIdx.x < samples) {
        const int64_t x = (int64_t)threadIdx.x * V / samples;
        const uint32_t k = (uint32_t)x - q[qs * x + 1] + 1;             // root + 1
        uint32_t h = (k * 2654435761u) >> 21;
        for (;;) {
            const uint32_t old = atomicCAS(&key[h], 0u, k);
            if (old == 0 || old == k) { atomicAdd(&num[h], 1u); break; }
            h = (h + 1) & (2 * kPick - 1);
        }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < 2 * kPick; i += kPick)
        if (key[i]) {
            const uint32_t p = atomicAdd(&nd, 1u);
            root[p] = key[i] - 1;
            freq[p] = num[i];
        }
    __syncthreads();
    if (threadIdx.x < nd) {
        const uint32_t f = freq[threadIdx.x];
        uint32_t rank = 0;
        for (uint32_t j = 0; j < nd; j += 4) {
            const uint4 g = *reinterpret_cast<const uint4*>(&freq[j]);
            rank += (g.x > f || (g.x == f && j < threadIdx.x)) + (g.y > f || (g.y == f && j + 1 < threadIdx.x)) +
                    (g.z > f || (g.z == f && j + 2 < threadIdx.x)) + (g.w > f || (g.w == f && j + 3 < threadIdx.x));
        }
        if (rank < (uint32_t)ncodes) rcode[root[threadIdx.x]] = rank + 1;
    }
}

// the packed table: word w holds the codes of vertices [w * kPer, (w + 1) * kPer)
template <int kPer>
__global__ void __launch_bounds__(256) k_codes(const uint32_t* q, int64_t qs, int32_t V, const uint32_t* rcode,
                                               uint32_t* code, int64_t words) {
    constexpr int kBits = 32 / kPer;
    GRID_LOOP(w, words) {
        uint32_t v = 0;
#pragma unroll
        for (int j = 0; j < kPer; j++) {
            const int64_t x = w * kPer + j;
            if (x < V) v |= rcode[(uint32_t)x - q[qs * x + 1]] << (j * kBits);
        }
        code[w] = v;
    }
}

template <int kPer>
__device__ __forceinline__ uint32_t code_of(const uint32_t* tab, uint32_t x) {
    constexpr int kBits = 32 / kPer;
    if constexpr (kPer == 2) return reinterpret_cast<const uint16_t*>(tab)[x];
    else if constexpr (kPer == 4) return reinterpret_cast<const uint8_t*>(tab)[x];
    else return (tab[x / kPer] >> ((x % kPer) * kBits)) & ((1u << kBits) - 1u);
}

// lanes [0, n) of a wavefront offer edges l[0..n); accepted ones go straight to
// the region (few are accepted after stage 2: one reservation per list)
__device__ __forceinline__ void offer_list(const DevBufs& B, int64_t cap, const int2* l, uint32_t n) {
    bool a1 = false, a2 = false;
    int2 e = make_int2(0, 0);
    uint64_t su = 0, sv = 0;
    const uint32_t lane = __lane_id();
    if (lane < n) {
        e = l[lane];
        su = ld2(B.state + B.qs * (int64_t)e.x);
        sv = ld2(B.state + B.qs * (int64_t)e.y);
    }
    offer_from(B.state, B.qs, lane < n, (uint32_t)e.x, (uint32_t)e.y, su, sv, a1, a2);
    for (int f = 0; f < 2; f++) {
        const bool a = f ? a2 : a1;
        const uint64_t m = __ballot(a);
        if (!m) continue;
        const int leader = __ffsll((unsigned long long)m) - 1;
        uint32_t base = 0;
        if ((int)lane == leader) base = atomicAdd(B.cnt + f, (uint32_t)__popcll(m));
        base = __shfl(base, leader);
        if (a) {
            const int64_t pos = (int64_t)base + lane_rank(m);
            if (pos >= cap) atomicOr(B.err, 2u);
            else B.cert[f ? cap - 1 - pos : pos] = e;
        }
    }
}

// lanes [0, n) append edges l[0..n) to out[]; past `room` they are only counted
__device__ __forceinline__ void append_list(int2* out, uint32_t* nout, uint32_t room, const int2* l, uint32_t n) {
    const uint32_t lane = __lane_id();
    uint32_t base = 0;
    if (lane == 0) base = atomicAdd(nout, n);
    base = __shfl(base, 0);
    if (lane < n && base + lane < room) out[base + lane] = l[lane];
}

// where k_filter's remaining edges go: the union-find (out null) or a list
struct Sink {
    int2* out;
    uint32_t* nout;
    uint32_t room;
};

typedef int edge2 __attribute__((ext_vector_type(4), aligned(8)));   // two edges, 8-byte aligned

// Stage 3: all rows that are not multiples of div + 1 (div = 0: all rows).  A wavefront takes 128
// edges (two per lane) at a time, kU such loads in flight; every wavefront
// keeps its own list, so the stream has no barrier.
//
// kItems: the list is a union of graphs whose edges start at whole rows;
// workgroup b takes the rows of item b that are not multiples of div + 1, with
// a table of its graph alone -- every component named by its root.
template <int kPer, bool kSplit, bool kList, bool kItems>
__global__ void __launch_bounds__(kFilterBlock) k_filter(DevBufs B, int64_t E, int32_t V, int64_t cap, uint32_t nsel,
                                                         uint32_t div, const uint32_t* code, int32_t words, Sink K,
                                                         const RowItem* items) {
    constexpr int kU = 4;
    static_assert(!kItems || kPer == 2, "a graph of a union has 16-bit codes");
    RowItem it{};
    if constexpr (kItems) it = items[blockIdx.x];
    auto drain = [&](const int2* l, uint32_t k) {
        if constexpr (kList) append_list(K.out, K.nout, K.room, l, k);
        else offer_list(B, cap, l, k);
    };
    extern __shared__ __align__(16) uint32_t lds[];
    uint32_t* tab = lds;
    if constexpr (kItems) {
        for (int32_t x = threadIdx.x; x < it.V; x += kFilterBlock) {
            const uint32_t d = B.state[B.qs * ((int64_t)it.base + x) + 1];
            reinterpret_cast<uint16_t*>(tab)[x] = (uint16_t)(x - (int32_t)d + 1);
        }
    } else {
        for (int32_t i = threadIdx.x; i < words / 4; i += kFilterBlock)
            reinterpret_cast<uint4*>(tab)[i] = reinterpret_cast<const uint4*>(code)[i];
    }
    __syncthreads();
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    int2* wl = reinterpret_cast<int2*>(lds + words) + wave * kListCap;
    uint32_t n = 0;                                                     // edges in the list (uniform)
    const int64_t units = (int64_t)(kItems ? it.r1 - it.r0 : nsel) * (kRow / 128);
    const int64_t stride = kItems ? kFilterWaves : (int64_t)gridDim.x * kFilterWaves;
    for (int64_t u = kItems ? wave : (int64_t)blockIdx.x * kFilterWaves + wave; u < units; u += stride * kU) {
        int2 e[kU][2];
        uint32_t have = 0;
#pragma unroll
        for (int j = 0; j < kU; j++) {
            const int64_t uu = u + j * stride;
            e[j][0] = e[j][1] = make_int2(0, 0);
            const uint32_t sel = (uint32_t)(uu >> 2);
            if (uu < units && !(kItems && (it.r0 + sel) % (div + 1) == 0)) {
                const int64_t i = (kItems ? (int64_t)(it.r0 + sel) : stage_row(sel, 1, div)) * kRow + (uu & 3) * 128 + 2 * lane;
                if (i + 1 < E) {
                    if constexpr (kSplit) {
                        e[j][0] = edge_at(B, i);
                        e[j][1] = edge_at(B, i + 1);
                    } else {
                        const edge2 w = *reinterpret_cast<const edge2*>(B.edges + i);
                        e[j][0] = make_int2(w.x, w.y);
                        e[j][1] = make_int2(w.z, w.w);
                    }
                    have |= 3u << (2 * j);
                } else if (i < E) {
                    e[j][0] = edge_at(B, i);
                    have |= 1u << (2 * j);
                }
            }
        }
#pragma unroll
        for (int j = 0; j < kU; j++) {
#pragma unroll
            for (int t = 0; t < 2; t++) {
                const uint32_t x = (uint32_t)e[j][t].x, y = (uint32_t)e[j][t].y;
                bool hard = false;
                if (have >> (2 * j + t) & 1u) {
                    if (kItems) {
                        // (-1: an id that was out of its graph's range)
                        const uint32_t a = x - (uint32_t)it.base, b = y - (uint32_t)it.base;
                        if (a < (uint32_t)it.V && b < (uint32_t)it.V) hard = code_of<kPer>(tab, a) != code_of<kPer>(tab, b);
                        else atomicOr(B.err, 1u);
                    } else if (x < (uint32_t)V && y < (uint32_t)V) {
                        const uint32_t cx = code_of<kPer>(tab, x), cy = code_of<kPer>(tab, y);
                        hard = cx != cy || cx == 0;
                    } else {
                        atomicOr(B.err, 1u);
                    }
                }
                const uint64_t m = __ballot(hard);
                if (m) {
                    if (hard) wl[n + lane_rank(m)] = e[j][t];
                    n += (uint32_t)__popcll(m);
                    __builtin_amdgcn_wave_barrier();       // written by the wavefront's lanes, read back by them
                    if (n >= 64) {
                        n -= 64;
                        drain(wl + n, 64);
                        __builtin_amdgcn_wave_barrier();
                    }
                }
            }
        }
    }
    if constexpr (kList) {
        // what is left in the lists: one reservation per workgroup (one per
        // wavefront, 4,096 on one address, took 30 us)
        __shared__ uint32_t left[kFilterWaves + 1];
        if (lane == 0) left[wave] = n;
        __syncthreads();
        if (threadIdx.x == 0) {
            uint32_t sum = 0;
            for (int w = 0; w < kFilterWaves; w++) {
                const uint32_t c = left[w];
                left[w] = sum;
                sum += c;
            }
            left[kFilterWaves] = sum ? atomicAdd(K.nout, sum) : 0u;
        }
        __syncthreads();
        const uint32_t base = left[kFilterWaves] + left[wave];
        if (lane < n && base + lane < K.room) K.out[base + lane] = wl[lane];
    } else if (n) {
        drain(wl, n);
    }
}

template <int kPer>
void launch_filter(const DevBufs& B, const Plan& P, uint32_t nsel, uint32_t div, const uint32_t* code, int grid,
                   const Sink& K, hipStream_t s) {
    const size_t lds = 4 * (size_t)P.code_words + kListBytes;
    auto k = K.out ? &k_filter<kPer, false, true, false>
                   : (B.edges2 && B.split < P.E ? &k_filter<kPer, true, false, false> : &k_filter<kPer, false, false, false>);
    hipLaunchKernelGGL(k, dim3(grid), dim3(kFilterBlock), lds, s, B, P.E, P.V, P.cap[0], nsel, div, code, P.code_words, K,
                       (const RowItem*)nullptr);
}

// f(integral constant) for the codes per word
template <class Fn>
void with_per(int32_t per, Fn f) {
    switch (per) {
        case 2: f(std::integral_constant<int, 2>()); break;
        case 4: f(std::integral_constant<int, 4>()); break;
        case 8: f(std::integral_constant<int, 8>()); break;
        case 16: f(std::integral_constant<int, 16>()); break;
        default: f(std::integral_constant<int, 32>()); break;
    }
}

template <int kPer>
hipError_t raise_lds() {
    std::vector<void (*)(DevBufs, int64_t, int32_t, int64_t, uint32_t, uint32_t, const uint32_t*, int32_t, Sink, const RowItem*)> ks{
        &k_filter<kPer, false, false, false>, &k_filter<kPer, true, false, false>, &k_filter<kPer, false, true, false>};
    if constexpr (kPer == 2) ks.push_back(&k_filter<2, false, false, true>);
    for (auto k : ks) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(k),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, kFilterLds - 256);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// codes for the largest components (where every root does not have one), then
// the packed table; word 1 of a vertex's state (q[qs * x + 1]) leads to its root
void launch_codes(const Plan& P, const uint32_t* q, int64_t qs, const FusedBufs& F, hipStream_t s, int* launches) {
    if (P.code_per > 2) {
        const int ncodes = (1 << (32 / P.code_per)) - 1;
        hipLaunchKernelGGL(k_pick, dim3(1), dim3(kPick), 0, s, q, qs, P.V, ncodes > 15 ? kPick : 256, ncodes, F.rcode);
        ++*launches;
    }
    with_per(P.code_per, [&](auto per) {
        hipLaunchKernelGGL(k_codes<decltype(per)::value>, dim3((unsigned)((P.code_words + 255) / 256)), dim3(256), 0, s, q, qs,
                           P.V, (const uint32_t*)F.rcode, F.code, (int64_t)P.code_words);
    });
    ++*launches;
}

// stage 3 over every row that is not a multiple of P.s2 (every row at all with
// a list as sink)
void launch_rest(const Plan& P, const DevBufs& B, const FusedBufs& F, const Sink& K, hipStream_t s) {
    const int64_t nrows = (P.E + kRow - 1) / kRow;
    const uint32_t nsel = (uint32_t)(K.out ? nrows : nrows - (nrows + P.s2 - 1) / P.s2);
    const uint32_t div = K.out ? 0u : (uint32_t)(P.s2 - 1);
    const int cus = g_cus > 0 ? g_cus : 256;
    // a wavefront takes at least four loads' worth of the list; two
    // workgroups share a CU where their tables allow it
    const int64_t units = (int64_t)nsel * (kRow / 128);
    const int per_cu = 4 * (int64_t)P.code_words + kListBytes <= kFilterLds / 2 ? 2 : 1;
    const int grid = (int)std::max<int64_t>(1, std::min<int64_t>((int64_t)cus * per_cu, (units + 4 * kFilterWaves - 1) / (4 * kFilterWaves)));
    with_per(P.code_per, [&](auto per) { launch_filter<decltype(per)::value>(B, P, nsel, div, F.code, grid, K, s); });
}

}  // namespace

// Strides and table of the plan's stages (E, V set).  Two stages past 3V edges:
// a merge's 3.98V edges over 10^5 vertices 94 us in one, 53 + 11 (compression)
// + 18 in two; 2.5V over 400,009 vertices 167 against 90 + 22 + 74 us.
void plan_fused(Plan& P) {
    const int64_t E = P.E, V = P.V;
    P.s1 = P.s2 = 1;
    if (E > 16 * V) {
        P.s2 = (int32_t)std::min<int64_t>(E / (8 * V), 1 << 20);
        P.s1 = 4 * P.s2;
    } else if (E > 3 * V) {
        P.s1 = P.s2 = (int32_t)std::max<int64_t>(2, E / (2 * V));
    }
    P.code_per = 0;
    P.code_words = 0;
    if (P.table && E > 16 * V && E >= (int64_t(1) << 19))
        for (int per : {2, 4, 8, 16, 32})
            if (4 * ((V + per - 1) / per) <= kTabBytes) {
                P.code_per = per;
                P.code_words = (int32_t)((((V + per - 1) / per) + 3) & ~int64_t(3));
                break;
            }
}

int fused_prepare() {
    static OncePerDevice once;
    const hipError_t e = once([] {
        for (hipError_t r : {raise_lds<2>(), raise_lds<4>(), raise_lds<8>(), raise_lds<16>(), raise_lds<32>()})
            if (r != hipSuccess) return r;
        return hipSuccess;
    });
    return e == hipSuccess ? BR_OK : hip_fail(e, "hipFuncSetAttribute(k_filter)");
}

void launch_fused_init(void* base, size_t bytes, int64_t* off, int64_t* cap, int64_t cap0, hipStream_t s) {
    const int64_t n16 = (int64_t)bytes / 16;
    hipLaunchKernelGGL(k_fused_init, dim3((unsigned)std::max<int64_t>(1, std::min<int64_t>((n16 + 255) / 256, 4096))),
                       dim3(256), 0, s, reinterpret_cast<uint4*>(base), n16, off, cap, cap0);
}

void launch_filter_rest(const Plan& P, const DevBufs& B, const FusedBufs& F, hipStream_t s) {
    launch_rest(P, B, F, Sink{}, s);
}

int launch_list_rest(const Plan& P, const DevBufs& B, const FusedBufs& F, uint32_t* g, int2* out, uint32_t* nout,
                     uint32_t room, hipStream_t s) {
    int launches = 2;
    hipLaunchKernelGGL(k_flatten1, dim3((unsigned)std::max<int64_t>(1, std::min<int64_t>(((int64_t)P.V + 255) / 256, 16384))),
                       dim3(256), 0, s, g, P.V, F.rcode, F.ncode, P.code_per == 2 ? 1 : 0);
    launch_codes(P, g - 1, 1, F, s, &launches);      // g's word is read as word 1
    launch_rest(P, B, F, Sink{out, nout, room}, s);
    return launches;
}

static void launch_flatten(const Plan& P, const DevBufs& B, uint32_t* rcode, uint32_t* ncode, hipStream_t s) {
    hipLaunchKernelGGL(k_flatten, dim3((unsigned)std::max<int64_t>(1, std::min<int64_t>(((int64_t)P.V + 255) / 256, 16384))),
                       dim3(256), 0, s, B.state, B.qs, P.V, rcode, ncode);
}

void launch_flatten(const Plan& P, const DevBufs& B, hipStream_t s) { launch_flatten(P, B, nullptr, nullptr, s); }

int launch_fused(const Plan& P, const DevBufs& B, const FusedBufs& F, hipStream_t s) {
    if (P.E == 0) return 0;
    int launches = 0;
    const int64_t nrows = (P.E + kRow - 1) / kRow;
    const int64_t m1 = (nrows + P.s1 - 1) / P.s1, m2 = (nrows + P.s2 - 1) / P.s2;
    const int cus = g_cus > 0 ? g_cus : 256;
    auto rows = [&](int64_t nsel, int32_t mul, uint32_t div, int64_t rpw_want) {
        if (nsel <= 0) return;
        const int32_t rpw = (int32_t)std::max<int64_t>(1, std::min<int64_t>(kMaxRows, rpw_want));
        hipLaunchKernelGGL(k_rows, dim3((unsigned)((nsel + rpw - 1) / rpw)), dim3(kRowBlock), 0, s, B, P.E, P.V, P.cap[0],
                           (uint32_t)nsel, mul, div, rpw);
        launches++;
    };
    auto flatten = [&](bool codes) {
        launch_flatten(P, B, codes ? F.rcode : nullptr, F.ncode, s);
        launches++;
    };
    // Most of stage 1 is accepted: as many workgroups as the chip holds at once before
    // a workgroup takes a second row (the chains of dependent reads decide, not the
    // launch).  Few of stage 2's edges are, and its workgroups wait for each other's
    // reservations, 12 ns each: half as many (dense 874 rows: 23.3 us with a workgroup
    // each, 19.2 so; large 3,130 rows: 64.4 us in threes, 48.3 in sevens).
    const auto spread = [&](int64_t nsel) { return nsel / (4 * cus); };
    const auto gathered = [&](int64_t nsel) { return (nsel + 2 * cus - 1) / (2 * cus); };
    rows(m1, P.s1, 0, spread(m1));
    if (P.s2 < P.s1) {
        flatten(false);
        rows(m2 - m1, P.s2, 3, gathered(m2 - m1));
    }
    if (P.s2 > 1) {
        const uint32_t nsel = (uint32_t)(nrows - m2), div = (uint32_t)(P.s2 - 1);
        flatten(P.code_per == 2);
        if (!P.table && F.items && P.s2 < P.s1) {
            // (after stage 1 alone too many edges still join components of F':
            // 405 us here for 9e6 edges over 560,000 vertices in 48 graphs)
            hipLaunchKernelGGL((k_filter<2, false, false, true>), dim3((unsigned)F.n_items), dim3(kFilterBlock),
                               4 * (size_t)F.item_words + kListBytes, s, B, P.E, P.V, P.cap[0], 0u, div,
                               (const uint32_t*)nullptr, F.item_words, Sink{}, F.items);
            return launches + 1;
        }
        if (P.code_per == 0) {
            rows(nsel, 1, div, spread(nsel));
            return launches;
        }
        launch_codes(P, B.state, B.qs, F, s, &launches);
        launch_filter_rest(P, B, F, s);
        launches++;
    }
    return launches;
}

}  // namespace br
