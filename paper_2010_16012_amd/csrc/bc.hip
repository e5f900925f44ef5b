// Brandes betweenness centrality on the BFS step (Sec. 3.5; Sec. 4.5
// listing), for a set of sources, in pushing and pulling forms.
//
// Per source s, level by level:
//  forward   sigma(w) = sum of sigma(v) over the edges v->w with
//            dist(w) = dist(v) + 1 (shortest-path counts);
//            push: frontier vertices claim unvisited targets (CAS on dist)
//            and add their sigma with FP64 atomics; pull: every unvisited
//            vertex sums sigma over its in-neighbours in the frontier and
//            writes only itself.
//  backward  delta(v) = sigma(v) * sum of (1 + delta(w)) / sigma(w) over the
//            edges v->w with dist(w) = dist(v) + 1, deepest level first;
//            push: each vertex of level l+1 adds to its predecessors with FP64
//            atomics; pull: each vertex of level l sums over its successors.
//  bc(v) += delta(v) for v != s.
// sigma, delta and bc are FP64 (path counts stay exact up to 2^53).  The
// vertices in BFS order (`order`) with per-level offsets give the frontiers
// of both phases.
//
// The kernels walk the internal (degree-ordered) adjacency, so the vertices
// every frontier reaches -- the hubs -- have the lowest ids.  The pushing
// kernels add contributions to the first kBcHot ids into per-workgroup LDS
// accumulators and hand each total to memory once per workgroup: without
// this, a hub's claim and its FP64 additions arrive from every one of its
// frontier neighbours and serialise on one address.
//
// Both passes pulling have kernels of their own, below, in which the sources of
// a batch share their walks; the rest of this comment is the other three forms.
//
// Sources run in batches of up to kBcBatch at once (the sources are
// independent, Sec. 4.5): every kernel has a grid row (blockIdx.y) per source
// of the batch, and each source owns a slab of the workspace (distances, path
// counts, dependencies, BFS order, level offsets).  The level bookkeeping of
// both passes is on the device: the last workgroup of a source's row to
// finish a level kernel records where its next level ends, whether it is
// empty, and (backward) which level comes next.  The host launches level
// kernels in batches (a source past its last level returns at once) and
// reads the states once per batch of forward levels; the backward levels
// follow without a read, and the dependencies are summed into bc in source
// order, without atomics.
#include <hip/hip_runtime.h>

#include <cstring>
#include <vector>

#include "pp_common.h"

namespace pp {

constexpr int kBcWaves = kBlock / kWave;
constexpr int32_t kBcHot = 4096;  // LDS-accumulated targets of the pushing kernels (32 KB of FP64)

constexpr int32_t kBcBatch = 32;  // sources processed together

// Level state of one source (level l is order[lvl_off[l], lvl_off[l + 1])).
struct BcState {
    int32_t l;         // level the next forward kernel expands
    int32_t done;      // set once a forward kernel found its next level empty
    int32_t depth;     // non-empty levels (valid once done)
    int32_t finished;  // workgroups of the running forward kernel that have finished
    int32_t bl;        // level the next backward kernel completes (-1: none left)
    int32_t bfinished; // workgroups of the running backward kernel that have finished
    int32_t pad[2];
};

// Pointers of source 0 of a batch; source s is `stride` bytes further on
// (see slab()).  st is an array over the batch.
struct BcArgs {
    int32_t n;
    int32_t hot;             // min(n, kBcHot)
    const int32_t* out_off;  // internal CSR (out-edges)
    const int32_t* out_idx;
    const int32_t* in_off;   // internal CSC (in-edges)
    const int32_t* in_idx;
    const int32_t* perm;     // internal -> caller id (nullable)
    const int32_t* iperm;    // caller -> internal id (nullable)
    int32_t* dist;
    double* sigma;
    double* delta;
    int32_t* order;    // vertices in BFS order
    int32_t* cnt;      // vertices in order so far
    int32_t* lvl_off;  // n + 2 entries
    BcState* st;
    size_t stride;     // bytes between the slabs of consecutive sources
    double* bc;        // caller ids
};

// The sources of a batch (caller ids), passed by value.
struct BcSources {
    int32_t s[kBcBatch];
};

template <typename T>
__device__ __forceinline__ T* shift(T* p, size_t bytes) {
    return reinterpret_cast<T*>(reinterpret_cast<char*>(p) + bytes);
}

// The arguments of source `s` of the batch.
__device__ __forceinline__ BcArgs slab(const BcArgs& a0, int32_t s) {
    BcArgs a = a0;
    const size_t b = (size_t)s * a0.stride;
    a.dist = shift(a0.dist, b);
    a.sigma = shift(a0.sigma, b);
    a.delta = shift(a0.delta, b);
    a.order = shift(a0.order, b);
    a.cnt = shift(a0.cnt, b);
    a.lvl_off = shift(a0.lvl_off, b);
    a.st = a0.st + s;
    return a;
}

__device__ __forceinline__ uint64_t bc_lanes_below(int lane) { return lane ? (~0ull >> (64 - lane)) : 0ull; }

// Appends the lanes with `mine` to order[] (one counter atomic per wave).
__device__ __forceinline__ void bc_append(const BcArgs& a, bool mine, int32_t w, int lane) {
    const uint64_t m = __ballot(mine);
    if (!m) return;
    int32_t base = 0;
    if (lane == 0) base = atomicAdd(a.cnt, (int32_t)__popcll(m));
    base = __shfl(base, 0);
    if (mine) a.order[base + __popcll(m & bc_lanes_below(lane))] = w;
}

// A wavefront's appends of a pushing level, collected in LDS: the counter is one
// address a source, and returning atomics on one address go one by one (a
// pushing level 206 -> 118 us at R-MAT 16 and 32 sources).
constexpr int kBcBuf = 2 * kWave;
struct BcBuf {
    int32_t* v;  // LDS, kBcBuf entries
    int32_t n;   // wave-uniform
};
__device__ __forceinline__ void bc_flush(const BcArgs& a, BcBuf& buf, int lane) {
    if (buf.n == 0) return;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    int32_t base = 0;
    if (lane == 0) base = atomicAdd(a.cnt, buf.n);
    base = __shfl(base, 0);
    for (int32_t i = lane; i < buf.n; i += kWave) a.order[base + i] = buf.v[i];
    buf.n = 0;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}
__device__ __forceinline__ void bc_collect(const BcArgs& a, BcBuf& buf, bool mine, int32_t w, int lane) {
    const uint64_t m = __ballot(mine);
    if (!m) return;
    const int32_t k = __popcll(m);
    if (buf.n + k > kBcBuf) bc_flush(a, buf, lane);
    if (mine) buf.v[buf.n + __popcll(m & bc_lanes_below(lane))] = w;
    buf.n += k;
}

// Position of lane `lane` of wavefront `gwave` (of `nwaves`) in pass `base`
// over a list: the 64 lanes of a wavefront take positions nwaves apart, so
// neighbouring list entries -- consecutive hubs in degree order, or hubs
// claimed together -- go to different wavefronts.
__device__ __forceinline__ int32_t spread(int32_t base, int lane, int32_t gwave, int32_t nwaves) {
    return base + lane * nwaves + gwave;
}

// Calls fn(valid, v, u) wave-collectively for every edge v->u of the rows
// (off/idx) of verts[0, count): 64 vertices per wave unit (spread over the
// list), rows of 64 or more edges walked by the whole wave, shorter ones
// enumerated densely.
template <typename Fn>
__device__ __forceinline__ void for_each_edge(const int32_t* verts, int32_t count, const int32_t* off,
                                              const int32_t* idx, Fn&& fn) {
    __shared__ int32_t s_start[kBcWaves][kWave];
    __shared__ int32_t s_rb[kBcWaves][kWave];
    __shared__ int32_t s_v[kBcWaves][kWave];
    const int lane = threadIdx.x & (kWave - 1);
    const int w = threadIdx.x / kWave;
    const int32_t gwave = blockIdx.x * kBcWaves + w;
    const int32_t nwaves = gridDim.x * kBcWaves;
    for (int32_t base = 0; base < count; base += nwaves * kWave) {
        const int32_t i = spread(base, lane, gwave, nwaves);
        const int32_t v = i < count ? verts[i] : -1;
        const int32_t rb = v >= 0 ? off[v] : 0, re = v >= 0 ? off[v + 1] : 0;
        const int32_t len = re - rb;
        uint64_t big = __ballot(len >= kWave);
        while (big) {
            const int src = __ffsll((long long)big) - 1;
            big &= big - 1;
            const int32_t bv = __shfl(v, src), bb = __shfl(rb, src), be = __shfl(re, src);
            for (slot_t j = (slot_t)bb + lane; j - lane < (slot_t)be; j += kWave)
                fn(j < (slot_t)be, bv, j < (slot_t)be ? idx[j] : -1);
        }
        const int32_t mine = len < kWave ? len : 0;
        int32_t incl = mine;
#pragma unroll
        for (int d = 1; d < kWave; d <<= 1) {
            const int32_t y = __shfl_up(incl, d);
            if (lane >= d) incl += y;
        }
        const int32_t total = __shfl(incl, kWave - 1);
        s_start[w][lane] = incl - mine;
        s_rb[w][lane] = rb;
        s_v[w][lane] = v;
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        for (int32_t k = 0; k < total; k += kWave) {
            const int32_t e = k + lane;
            int32_t pv = -1, u = -1;
            if (e < total) {
                int lo = 0, hi = kWave;  // last lane whose range starts at or before e
                while (hi - lo > 1) {
                    const int mid = (lo + hi) >> 1;
                    if (s_start[w][mid] <= e) lo = mid;
                    else hi = mid;
                }
                pv = s_v[w][lo];
                u = idx[s_rb[w][lo] + (e - s_start[w][lo])];
            }
            fn(e < total, pv, u);
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
}

// Sum of val(u) over the row [rb, re) of each lane's vertex (lanes with
// `own`), in stored order per lane; rows of 32 or more entries are summed by
// the wave (lane-strided, then a fixed shuffle tree).  Wave-collective.
constexpr int kBcU = 8;  // independent index loads in flight per lane

template <typename Val>
__device__ __forceinline__ double row_sum(bool own, int32_t rb, int32_t re, const int32_t* idx, int lane,
                                          Val&& val) {
    double acc = 0.0;
    const bool coop = own && (re - rb) >= 32;
    uint64_t big = __ballot(coop);
    while (big) {
        const int src = __ffsll((long long)big) - 1;
        big &= big - 1;
        const int32_t bb = __shfl(rb, src), be = __shfl(re, src);
        double t = 0.0;
        for (slot_t j0 = (slot_t)bb + lane; j0 < (slot_t)be; j0 += kBcU * kWave) {
            int32_t ii[kBcU];
#pragma unroll
            for (int k = 0; k < kBcU; ++k) ii[k] = slot_in(j0, k * kWave, be) ? idx[j0 + k * kWave] : -1;
#pragma unroll
            for (int k = 0; k < kBcU; ++k)
                if (ii[k] >= 0) t += val(ii[k]);
        }
#pragma unroll
        for (int d = 32; d > 0; d >>= 1) t += __shfl_xor(t, d);
        if (lane == src) acc = t;
    }
    if (own && !coop) {
        for (slot_t j0 = rb; j0 < (slot_t)re; j0 += kBcU) {
            int32_t ii[kBcU];
#pragma unroll
            for (int k = 0; k < kBcU; ++k) ii[k] = slot_in(j0, k, re) ? idx[j0 + k] : -1;
#pragma unroll
            for (int k = 0; k < kBcU; ++k)
                if (ii[k] >= 0) acc += val(ii[k]);
        }
    }
    return acc;
}

__global__ void k_bc_init(BcArgs a0, BcSources src) {
    const BcArgs a = slab(a0, blockIdx.y);
    const int32_t s_user = src.s[blockIdx.y];
    const int32_t s = a.iperm ? a.iperm[s_user] : s_user;
    for (int32_t v = blockIdx.x * blockDim.x + threadIdx.x; v < a.n; v += gridDim.x * blockDim.x) {
        a.dist[v] = v == s ? 0 : -1;
        a.sigma[v] = v == s ? 1.0 : 0.0;
        a.delta[v] = 0.0;
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        a.order[0] = s;
        *a.cnt = 1;
        *a.st = BcState{0, 0, 0, 0, -1, 0, {0, 0}};
        a.lvl_off[0] = 0;
        a.lvl_off[1] = 1;
    }
}

__global__ void k_bc_zero(int32_t n, double* bc) {
    for (int32_t v = blockIdx.x * blockDim.x + threadIdx.x; v < n; v += gridDim.x * blockDim.x) bc[v] = 0.0;
}

// Is this workgroup the last of its source's row to finish the kernel?
// (Every other one has then read the state.)  Workgroup-collective.
// No device-wide fence is needed (one would write back the whole L2 per
// workgroup): the appends are returning atomics on the counter, complete
// before the barrier, so the last workgroup's atomic read of the counter sees
// them all; what it writes is read by later kernels only.
__device__ __forceinline__ bool bc_last_group(int32_t* finished) {
    __shared__ int32_t s_last;
    __syncthreads();
    if (threadIdx.x == 0) s_last = atomicAdd(finished, 1) == (int32_t)gridDim.x - 1;
    __syncthreads();
    return s_last != 0;
}

// End of a forward level kernel: the last workgroup records the end of level
// l + 1 and whether it is empty (then the backward pass starts at the second
// deepest level), and advances the level.  Workgroup-collective.
__device__ __forceinline__ void bc_level_end(const BcArgs& a, int32_t l) {
    if (bc_last_group(&a.st->finished) && threadIdx.x == 0) {
        const int32_t c = atomicAdd(a.cnt, 0);
        a.lvl_off[l + 2] = c;
        if (c == a.lvl_off[l + 1]) {
            a.st->done = 1;
            a.st->depth = l + 1;
            a.st->bl = l - 1;
        }
        a.st->l = l + 1;
        a.st->finished = 0;
    }
}

// End of a backward level kernel: the last workgroup moves to the level above.
__device__ __forceinline__ void bc_back_end(const BcArgs& a, int32_t l) {
    if (bc_last_group(&a.st->bfinished) && threadIdx.x == 0) {
        a.st->bl = l - 1;
        a.st->bfinished = 0;
    }
}

// Zeroes the workgroup's hot accumulators.  Workgroup-collective.
__device__ __forceinline__ void hot_zero(double* s_acc, int32_t hot) {
    for (int32_t i = threadIdx.x; i < hot; i += blockDim.x) s_acc[i] = 0.0;
    __syncthreads();
}

// Forward, pushing: the frontier (level l) expands along out-edges.
__global__ __launch_bounds__(kBlock) void k_bc_fwd_push(BcArgs a0) {
    __shared__ double s_acc[kBcHot];
    const BcArgs a = slab(a0, blockIdx.y);
    const BcState st = *a.st;
    if (st.done) return;
    const int32_t l = st.l, lo = a.lvl_off[l], hi = a.lvl_off[l + 1];
    const int lane = threadIdx.x & (kWave - 1);
    __shared__ int32_t s_buf[kBcWaves][kBcBuf];
    BcBuf buf{s_buf[threadIdx.x / kWave], 0};
    hot_zero(s_acc, a.hot);
    for_each_edge(a.order + lo, hi - lo, a.out_off, a.out_idx, [&](bool valid, int32_t v, int32_t u) {
        bool claimed = false;
        if (valid) {
            if (u < a.hot) {
                unsafeAtomicAdd(&s_acc[u], a.sigma[v]);
            } else {
                int32_t d = a.dist[u];
                if (d == -1) {
                    d = atomicCAS(&a.dist[u], -1, l + 1);
                    claimed = d == -1;
                    if (claimed) d = l + 1;
                }
                if (d == l + 1) unsafeAtomicAdd(&a.sigma[u], a.sigma[v]);
            }
        }
        bc_collect(a, buf, claimed, u, lane);
    });
    __syncthreads();
    // hot targets this workgroup reached: a target with a contribution is on
    // level l + 1 exactly when it had no distance before this level
    for (int32_t base = threadIdx.x - lane; base < a.hot; base += blockDim.x) {
        const int32_t u = base + lane;
        const double sum = u < a.hot ? s_acc[u] : 0.0;
        bool claimed = false;
        if (sum != 0.0) {
            int32_t d = a.dist[u];
            if (d == -1) {
                d = atomicCAS(&a.dist[u], -1, l + 1);
                claimed = d == -1;
                if (claimed) d = l + 1;
            }
            if (d == l + 1) unsafeAtomicAdd(&a.sigma[u], sum);
        }
        bc_collect(a, buf, claimed, u, lane);
    }
    bc_flush(a, buf, lane);
    bc_level_end(a, l);
}

// Forward, pulling: every unvisited vertex sums sigma over its in-neighbours
// of level l; found vertices take level l+1.
__global__ __launch_bounds__(kBlock) void k_bc_fwd_pull(BcArgs a0) {
    const BcArgs a = slab(a0, blockIdx.y);
    const BcState st = *a.st;
    if (st.done) return;
    const int32_t l = st.l;
    const int lane = threadIdx.x & (kWave - 1);
    const int32_t gwave = blockIdx.x * kBcWaves + threadIdx.x / kWave, nwaves = gridDim.x * kBcWaves;
    for (int32_t base = 0; base < a.n; base += nwaves * kWave) {
        const int32_t w = spread(base, lane, gwave, nwaves);
        const bool own = w < a.n && a.dist[w] == -1;
        const int32_t rb = own ? a.in_off[w] : 0, re = own ? a.in_off[w + 1] : 0;
        const double acc = row_sum(own, rb, re, a.in_idx, lane,
                                   [&](int32_t v) { return a.dist[v] == l ? a.sigma[v] : 0.0; });
        const bool found = own && acc > 0.0;
        if (found) {
            a.dist[w] = l + 1;
            a.sigma[w] = acc;
        }
        bc_append(a, found, w, lane);
    }
    bc_level_end(a, l);
}

// Backward, pushing: every vertex w of level l+1 adds sigma(v) (1 + delta(w))
// / sigma(w) to each predecessor v (level l); hot predecessors collect the sum
// of (1 + delta(w)) / sigma(w) in LDS first.
__global__ __launch_bounds__(kBlock) void k_bc_bwd_push(BcArgs a0) {
    __shared__ double s_acc[kBcHot];
    const BcArgs a = slab(a0, blockIdx.y);
    const int32_t l = a.st->bl;
    if (l < 0) return;
    const int32_t lo = a.lvl_off[l + 1], hi = a.lvl_off[l + 2];
    const int lane = threadIdx.x & (kWave - 1);
    hot_zero(s_acc, a.hot);
    for_each_edge(a.order + lo, hi - lo, a.in_off, a.in_idx, [&](bool valid, int32_t w, int32_t v) {
        if (valid && a.dist[v] == l) {
            const double c = (1.0 + a.delta[w]) / a.sigma[w];
            if (v < a.hot) unsafeAtomicAdd(&s_acc[v], c);
            else unsafeAtomicAdd(&a.delta[v], a.sigma[v] * c);
        }
    });
    __syncthreads();
    for (int32_t base = threadIdx.x - lane; base < a.hot; base += blockDim.x) {
        const int32_t v = base + lane;
        const double sum = v < a.hot ? s_acc[v] : 0.0;
        if (sum != 0.0) unsafeAtomicAdd(&a.delta[v], a.sigma[v] * sum);
    }
    bc_back_end(a, l);
}

// Backward, pulling: every vertex v of level l sums over its successors
// (level l+1) and writes delta(v).
__global__ __launch_bounds__(kBlock) void k_bc_bwd_pull(BcArgs a0) {
    const BcArgs a = slab(a0, blockIdx.y);
    const int32_t l = a.st->bl;
    if (l < 0) return;
    const int32_t lo = a.lvl_off[l], hi = a.lvl_off[l + 1];
    const int lane = threadIdx.x & (kWave - 1);
    const int32_t gwave = blockIdx.x * kBcWaves + threadIdx.x / kWave, nwaves = gridDim.x * kBcWaves;
    for (int32_t base = lo; base < hi; base += nwaves * kWave) {
        const int32_t i = spread(base, lane, gwave, nwaves);
        const bool own = i < hi;
        const int32_t v = own ? a.order[i] : 0;
        const int32_t rb = own ? a.out_off[v] : 0, re = own ? a.out_off[v + 1] : 0;
        const double acc = row_sum(own, rb, re, a.out_idx, lane, [&](int32_t w) {
            return a.dist[w] == l + 1 ? (1.0 + a.delta[w]) / a.sigma[w] : 0.0;
        });
        if (own) a.delta[v] = a.sigma[v] * acc;
    }
    bc_back_end(a, l);
}

// bc(v) += delta_s(v) over the batch's sources s != v, in source order.
__global__ void k_bc_acc(BcArgs a0, BcSources src, int32_t count) {
    for (int32_t v = blockIdx.x * blockDim.x + threadIdx.x; v < a0.n; v += gridDim.x * blockDim.x) {
        const int32_t vu = a0.perm ? a0.perm[v] : v;
        double acc = 0.0;
        for (int32_t s = 0; s < count; ++s)
            if (src.s[s] != vu) acc += shift(a0.delta, (size_t)s * a0.stride)[v];
        a0.bc[vu] += acc;
    }
}

// ------------------------------------------- pulling levels of a whole batch
// Pulled in both directions, the sources of a batch share their walks of the
// adjacency.  Bit s of a vertex's word says whether the vertex is on the
// level at hand of source s, so one gather of four bytes an edge answers for
// all of them, and sigma lies source-minor (a line of KP doubles a vertex),
// so the values of the edges that count are gathered as whole lines, a lane
// a source.  (The kernels above read a distance per edge and source: 64
// million gathers a level at R-MAT 16 and 32 sources.)  64 sources there went
// from 3,040 to 710 us, 32 at R-MAT 20 from 20.6 to 4.7 ms; a full level takes 58 us for 512 MB of lines (9 TB/s,
// the caches' rate: the 16 MB of sigma are past an L2), a nearly empty one 6 to
// 17 us of load latency.  Loading a lane's value only where its bit is set took
// a quarter longer, kBcEdges at 128 and 512 4% and 19%, loading ahead what the
// ends of the rows need 3% (10% at R-MAT 20).
//
// A wavefront takes up to kBcRows consecutive rows of up to kBcEdges edges
// together: their ids are loaded at once, then their words; the edges that
// count go to a list in LDS in slot order, which the lane groups walk with
// kBcU lines in flight.  Heavier rows are units of their own (k_bc_units),
// cut at kBcEdges, whose partial sums the last wavefront to finish adds up in
// order, so every sum has a fixed order.  Levels are common to the batch: a
// source with fewer has no bits on the deeper ones.
constexpr int kBcRows = 8;
constexpr int kBcEdges = 256;
constexpr int kBcWin = kBcEdges / kWave;

// x: first row; y: -1 for a whole row, else pieces of it; z: piece;
// w: the row's first partial sum
typedef int4 BcUnit;

struct BcPullState {
    int32_t any[3];  // level l reached: any[l % 3]
    int32_t depth;   // non-empty levels found by the forward kernels so far
    int32_t units[2], parts[2];  // of the in-rows, out-rows
};

struct BcPull {
    int32_t n;
    uint32_t all;        // a bit for every source
    const int32_t* off;  // rows of the direction at hand
    const int32_t* idx;
    const BcUnit* units;
    int32_t side;        // 0: in-rows, 1: out-rows
    double* val;         // [n][KP] sigma; (1 + delta) / sigma once a level is complete backwards
    int32_t* dist;       // [n][KP], where vis has the bit
    uint32_t* vis;       // visited, a bit per source
    uint32_t* sig;       // bit d % 32: some source has the vertex at distance d
    const uint32_t* fm;  // on the level the sums come from (NULL: no vertex is)
    uint32_t* fn;        // on the level they make
    double* part;        // partial sums of cut rows [.][KP]
    int32_t* arrived;    // pieces of a cut row that are done (at the row's first partial sum)
    BcPullState* st;
    const int32_t* perm;
    double* bc;
    int32_t share;       // wavefronts to 64 light rows: 1, 2, 4 or 8
};

// Units of the rows too heavy to share a wavefront: those of each aligned
// group of kBcRows with more than kBcEdges edges together.
__global__ __launch_bounds__(kBlock) void k_bc_units(int32_t n, const int32_t* __restrict__ off, BcUnit* units,
                                                     int32_t* arrived, int32_t* n_units, int32_t* n_parts) {
    __shared__ int32_t s_units, s_parts, s_ubase, s_pbase;
    if (threadIdx.x == 0) s_units = s_parts = 0;
    __syncthreads();
    const int32_t v = blockIdx.x * blockDim.x + threadIdx.x;
    const int32_t d = v < n ? off[v + 1] - off[v] : 0;
    int64_t sum = d;
#pragma unroll
    for (int k = 1; k < kBcRows; k <<= 1) sum += __shfl_xor(sum, k);
    const bool heavy = v < n && sum > kBcEdges;
    const int32_t pieces = heavy ? max(1, (int32_t)(((int64_t)d + kBcEdges - 1) / kBcEdges)) : 0;
    const int32_t parts = pieces > 1 ? pieces : 0;
    const int32_t ua = pieces ? atomicAdd(&s_units, pieces) : 0;
    const int32_t pa = parts ? atomicAdd(&s_parts, parts) : 0;
    __syncthreads();
    if (threadIdx.x == 0) {
        s_ubase = s_units ? atomicAdd(n_units, s_units) : 0;
        s_pbase = s_parts ? atomicAdd(n_parts, s_parts) : 0;
    }
    __syncthreads();
    for (int32_t k = 0; k < pieces; ++k)
        units[s_ubase + ua + k] = make_int4(v, parts ? pieces : -1, k, s_pbase + pa);
    if (parts) arrived[s_pbase + pa] = 0;
}

// Level 0 of a batch.
template <int KP>
__global__ void k_bc_begin(BcPull a, BcSources src, int32_t count, const int32_t* __restrict__ iperm) {
    __shared__ int32_t s_src[kBcBatch];
    if ((int32_t)threadIdx.x < count) s_src[threadIdx.x] = iperm ? iperm[src.s[threadIdx.x]] : src.s[threadIdx.x];
    __syncthreads();
    for (int32_t v = blockIdx.x * blockDim.x + threadIdx.x; v < a.n; v += gridDim.x * blockDim.x) {
        uint32_t m = 0;
        for (int32_t s = 0; s < count; ++s) {
            if (s_src[s] != v) continue;
            m |= 1u << s;
            a.val[(size_t)v * KP + s] = 1.0;
            a.dist[(size_t)v * KP + s] = 0;
        }
        a.vis[v] = m;
        a.fn[v] = m;
        a.sig[v] = m ? 1u : 0u;
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        a.st->any[0] = 1;
        a.st->any[1] = a.st->any[2] = 0;
        a.st->depth = 0;
    }
}

// A wavefront's LDS.
struct BcWave {
    double acc[kBcRows][kWave];  // a row's sum, per lane
    int32_t id[kBcEdges];        // edges that count, in slot order
    uint32_t mask[kBcEdges];
    uint8_t row[kBcEdges];
};

__device__ __forceinline__ void bc_wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Sums val over the slots [eb, ee) (at most kBcEdges) of nr rows: rb (lanes
// 0..nr-1) is where the lane's row begins, need the sources it wants.
// Leaves w.acc[r][lane]; wave-collective.
template <int KP>
__device__ __forceinline__ void bc_sums(const BcPull& a, BcWave& w, int32_t eb, int32_t ee, int nr, int32_t rb,
                                        uint32_t need, int lane) {
    constexpr int G = kWave / KP;
    const int s = lane & (KP - 1), grp = lane / KP;
    for (int r = 0; r < nr; ++r) w.acc[r][lane] = 0.0;
    if (ee <= eb || !a.fm) {
        bc_wave_sync();
        return;
    }
    int32_t id[kBcWin];
    uint32_t m[kBcWin];
#pragma unroll
    for (int k = 0; k < kBcWin; ++k) id[k] = a.idx[eb + min(k * kWave + lane, ee - eb - 1)];
#pragma unroll
    for (int k = 0; k < kBcWin; ++k) m[k] = a.fm[id[k]];
    int32_t begin[kBcRows];
#pragma unroll
    for (int r = 1; r < kBcRows; ++r) begin[r] = r < nr ? __builtin_amdgcn_readlane(rb, r) - eb : INT32_MAX;
    int32_t total = 0;
#pragma unroll
    for (int k = 0; k < kBcWin; ++k) {
        const int32_t slot = k * kWave + lane;  // from eb
        int row = 0;
#pragma unroll
        for (int r = 1; r < kBcRows; ++r) row += slot >= begin[r];
        const uint32_t want = (uint32_t)__shfl((int)need, row);
        const uint32_t mm = slot < ee - eb ? m[k] & want : 0u;
        const uint64_t bal = __ballot(mm != 0);
        if (mm) {
            const int32_t at = total + __popcll(bal & bc_lanes_below(lane));
            w.id[at] = id[k];
            w.mask[at] = mm;
            w.row[at] = (uint8_t)row;
        }
        total += __popcll(bal);
    }
    bc_wave_sync();
    double acc = 0.0;
    int cur = -1;
    for (int32_t i0 = grp; i0 < total; i0 += kBcU * G) {
        double v[kBcU];
        uint32_t mk[kBcU];
        int row[kBcU];
#pragma unroll
        for (int k = 0; k < kBcU; ++k) {
            const int32_t i = i0 + k * G, c = min(i, total - 1);
            mk[k] = i < total ? w.mask[c] : 0u;
            row[k] = w.row[c];
            v[k] = a.val[(size_t)w.id[c] * KP + s];  // read only where the bit is set
        }
#pragma unroll
        for (int k = 0; k < kBcU; ++k) {
            if (row[k] != cur && i0 + k * G < total) {
                if (cur >= 0) w.acc[cur][lane] = acc;
                acc = 0.0;
                cur = row[k];
            }
            acc += (mk[k] >> s) & 1u ? v[k] : 0.0;
        }
    }
    if (cur >= 0) w.acc[cur][lane] = acc;
    bc_wave_sync();
}

// The row's sum `acc` of source s is complete (a lane group a row; `mine`:
// the group has a row; need: the sources the row wants).  Wave-collective.
template <int KP, bool FWD>
__device__ __forceinline__ uint32_t bc_finish(const BcPull& a, int32_t l, bool mine, int32_t row, uint32_t need,
                                              double acc, int lane) {
    const int s = lane & (KP - 1), grp = lane / KP;
    constexpr uint32_t kBits = KP == 32 ? 0xFFFFFFFFu : (1u << KP) - 1u;
    const bool on = mine && ((need >> s) & 1u);
    const size_t at = (size_t)row * KP + s;
    if constexpr (FWD) {
        const bool found = on && acc > 0.0;
        const uint32_t m = (uint32_t)(__ballot(found) >> (grp * KP)) & kBits;
        if (found) {
            a.val[at] = acc;
            a.dist[at] = l + 1;
        }
        if (mine && s == 0) {
            a.fn[row] = m;
            if (m) {
                a.vis[row] = (a.all & ~need) | m;
                a.sig[row] |= 1u << ((l + 1) & 31);
            }
        }
        return mine ? m : 0u;
    } else {
        double d = 0.0;
        if (on) {
            const double sigma = a.val[at];
            d = sigma * acc;
            a.val[at] = (1.0 + d) / sigma;
        }
#pragma unroll
        for (int k = KP / 2; k > 0; k >>= 1) d += __shfl_xor(d, k);
        if (mine && s == 0) {
            a.fn[row] = need;
            if (need) {
                const int32_t u = a.perm ? a.perm[row] : row;
                a.bc[u] += d;
            }
        }
        return 0u;
    }
}

// One level of all sources: forwards, vertices not yet visited sum sigma over
// their in-neighbours on level l and join level l + 1; backwards, vertices on
// level l sum over their successors on level l + 1.
template <int KP, bool FWD>
__global__ __launch_bounds__(kBlock) void k_bc_level(BcPull a, int32_t l) {
    __shared__ BcWave s_wave[kBcWaves];
    constexpr int G = kWave / KP;
    constexpr uint32_t kBits = KP == 32 ? 0xFFFFFFFFu : (1u << KP) - 1u;
    const int lane = threadIdx.x & (kWave - 1);
    const int s = lane & (KP - 1), grp = lane / KP;
    BcWave& w = s_wave[threadIdx.x / kWave];
    if constexpr (FWD) {
        const int32_t any = a.st->any[l % 3];
        if (blockIdx.x == 0 && threadIdx.x == 0) {
            a.st->any[(l + 2) % 3] = 0;
            if (any) a.st->depth = l + 1;
        }
        if (!any) return;
    }
    const int32_t gwave = blockIdx.x * kBcWaves + threadIdx.x / kWave, nwaves = gridDim.x * kBcWaves;
    uint32_t found = 0;
    // heavy rows
    const int32_t nu = a.st->units[a.side];
    for (int32_t i = gwave; i < nu; i += nwaves) {
        const BcUnit u = a.units[i];
        const int32_t row = u.x;
        const int32_t rb = a.off[row], re = a.off[row + 1];
        uint32_t need = a.vis[row];
        if constexpr (FWD) {
            need = a.all & ~need;
        } else {
            if ((a.sig[row] >> (l & 31)) & 1u) need &= (uint32_t)__ballot(a.dist[(size_t)row * KP + s] == l) & kBits;
            else need = 0;
        }
        need = (uint32_t)__builtin_amdgcn_readfirstlane((int)need);
        if (need == 0) {
            if (u.z == 0 && lane == 0) a.fn[row] = 0;
            continue;
        }
        const int32_t eb = u.y > 0 ? rb + u.z * kBcEdges : rb;
        const int32_t ee = u.y > 0 && u.z + 1 < u.y ? eb + kBcEdges : re;
        bc_sums<KP>(a, w, eb, ee, 1, rb, need, lane);
        double acc = 0.0;
#pragma unroll
        for (int g = 0; g < G; ++g) acc += w.acc[0][g * KP + s];
        bc_wave_sync();
        if (u.y > 0) {
            // the partial sum is at memory before the piece counts as done:
            // the exchange returns (no fence, which would write back the L2)
            double* p = a.part + (size_t)u.w * KP;
            if (grp == 0) {
                unsigned long long was = atomicExch(reinterpret_cast<unsigned long long*>(p + (size_t)u.z * KP + s),
                                                    (unsigned long long)__double_as_longlong(acc));
                asm volatile("" ::"v"(was) : "memory");
            }
            __builtin_amdgcn_wave_barrier();
            int32_t was = 0;
            if (lane == 0) was = atomicAdd(&a.arrived[u.w], 1);
            if (__builtin_amdgcn_readfirstlane(was) != u.y - 1) continue;
            if (lane == 0) a.arrived[u.w] = 0;
            acc = 0.0;
            for (int32_t i0 = grp; i0 < u.y; i0 += kBcU * G) {
                double v[kBcU];
#pragma unroll
                for (int k = 0; k < kBcU; ++k)
                    v[k] = __hip_atomic_load(p + (size_t)min(i0 + k * G, u.y - 1) * KP + s, __ATOMIC_RELAXED,
                                             __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
                for (int k = 0; k < kBcU; ++k) acc += i0 + k * G < u.y ? v[k] : 0.0;
            }
#pragma unroll
            for (int k = KP; k < kWave; k <<= 1) acc += __shfl_xor(acc, k);
        }
        found |= bc_finish<KP, FWD>(a, l, grp == 0, row, need, acc, lane);
    }
    // the other rows: 64 looked at together, of which the wavefront takes
    // every `share`-th group (on small graphs the groups of one wavefront, a
    // few microseconds each, would be the longest chain of the launch)
    const int32_t blocks = (a.n + kWave - 1) / kWave;
    for (int64_t item = nwaves - 1 - gwave; item < (int64_t)blocks * a.share; item += nwaves) {
        const int32_t b = (int32_t)(item / a.share), part = (int32_t)(item % a.share);
        const int32_t v = b * kWave + lane;
        const bool in = v < a.n;
        const int32_t rb = in ? a.off[v] : 0, re = in ? a.off[v + 1] : 0;
        uint32_t need = in ? a.vis[v] : 0u;
        if constexpr (FWD) need = in ? a.all & ~need : 0u;
        else if (!(in && ((a.sig[v] >> (l & 31)) & 1u))) need = 0u;
        int64_t sum = re - rb;
#pragma unroll
        for (int k = 1; k < kBcRows; k <<= 1) sum += __shfl_xor(sum, k);
        const bool light = in && sum <= kBcEdges && (lane / kBcRows) % a.share == part;
        uint64_t todo = __ballot(light && need != 0);
        // rows of a group that nobody wants
        if (light && !((todo >> (lane & ~(kBcRows - 1))) & ((1ull << kBcRows) - 1))) a.fn[v] = 0;
        while (todo) {
            const int first = (__ffsll((long long)todo) - 1) & ~(kBcRows - 1);
            todo &= ~(((1ull << kBcRows) - 1) << first);
            const int32_t r0 = b * kWave + first;
            const int nr = min(kBcRows, a.n - r0);
            // lanes 0..nr-1 take over the group's rows
            const int32_t gb = __shfl(rb, (first + lane) & (kWave - 1));
            uint32_t gn = (uint32_t)__shfl((int)need, (first + lane) & (kWave - 1));
            const int32_t eb = __builtin_amdgcn_readlane(rb, first);
            const int32_t ee = __builtin_amdgcn_readlane(re, first + nr - 1);
            if constexpr (!FWD) {
                int32_t d[kBcRows];  // of row k + grp
#pragma unroll
                for (int k = 0; k < kBcRows; k += G) d[k] = a.dist[(size_t)(r0 + min(k + grp, nr - 1)) * KP + s];
                uint32_t at = 0;
#pragma unroll
                for (int k = 0; k < kBcRows; k += G) {
                    const uint64_t bal = __ballot(d[k] == l);
                    if (lane >= k && lane < k + G) at = (uint32_t)(bal >> ((lane - k) * KP)) & kBits;
                }
                gn &= at;
                if (!__ballot(lane < nr && gn != 0)) {
                    if (lane < nr) a.fn[r0 + lane] = 0;
                    continue;
                }
            }
            bc_sums<KP>(a, w, eb, ee, nr, gb, lane < nr ? gn : 0u, lane);
#pragma unroll
            for (int k = 0; k < kBcRows; k += G) {
                if (k >= nr) break;
                const int r = min(k + grp, nr - 1);
                double acc = 0.0;
#pragma unroll
                for (int g = 0; g < G; ++g) acc += w.acc[r][g * KP + s];
                found |= bc_finish<KP, FWD>(a, l, k + grp < nr, r0 + r, (uint32_t)__shfl((int)gn, r), acc, lane);
            }
            bc_wave_sync();
        }
    }
    if constexpr (FWD) {
        if (__ballot(found != 0) && lane == 0) a.st->any[(l + 1) % 3] = 1;
    }
}

// One source's slab; the workspace holds the batch's states, then up to
// kBcBatch slabs.
struct BcLayout {
    size_t dist, sigma, delta, order, cnt, lvl_off, slab;
};

static BcLayout bc_layout(int32_t n) {
    BcLayout L{};
    size_t p = 0;
    auto take = [&](size_t bytes) {
        size_t at = p;
        p = align_up(p + bytes, 256);
        return at;
    };
    L.dist = take((size_t)n * 4);
    L.sigma = take((size_t)n * 8);
    L.delta = take((size_t)n * 8);
    L.order = take((size_t)n * 4);
    L.cnt = take(4);
    L.lvl_off = take(((size_t)n + 2) * 4);
    L.slab = p;
    return L;
}

constexpr size_t kBcStates = (sizeof(BcState) * kBcBatch + 255) / 256 * 256;

// Workspace of the batch's pulling levels, kp columns a vertex.  A row has at
// most 1 + d / kBcEdges units, a cut one (d > kBcEdges) at most 2 d / kBcEdges pieces.
struct BcPullLayout {
    size_t st, val, dist, vis, sig, f0, f1, units0, units1, part, arrived, total;
};

static BcPullLayout bc_pull_layout(int64_t n, int64_t nnz, int kp, bool symmetric) {
    BcPullLayout L{};
    size_t p = 0;
    auto take = [&](size_t bytes) {
        size_t at = p;
        p = align_up(p + bytes, 256);
        return at;
    };
    const size_t units = (size_t)std::min(n + nnz / kBcEdges + 1, n / kBcRows + 9 * (nnz / kBcEdges) + 16);
    const size_t parts = (size_t)(2 * (nnz / kBcEdges) + 2);
    L.st = take(sizeof(BcPullState));
    L.val = take((size_t)n * kp * 8);
    L.dist = take((size_t)n * kp * 4);
    L.vis = take((size_t)n * 4);
    L.sig = take((size_t)n * 4);
    L.f0 = take((size_t)n * 4);
    L.f1 = take((size_t)n * 4);
    L.units0 = take(units * sizeof(BcUnit));
    L.units1 = symmetric ? L.units0 : take(units * sizeof(BcUnit));
    L.part = take(parts * kp * 8);
    L.arrived = take(parts * 4);
    L.total = p;
    return L;
}

// Both passes pulling, for sources in batches of up to KP.
template <int KP>
static pp_status bc_pull_run(pp_graph g, const BcPullLayout& L, int32_t num_sources, const int32_t* sources,
                             double* bc, char* ws, hipStream_t st) {
    const int32_t n = g->d.n;
    const bool symmetric = g->d.csr_off == g->d.csc_off && g->d.csr_idx == g->d.csc_idx;
    BcPull a;
    a.n = n;
    a.val = reinterpret_cast<double*>(ws + L.val);
    a.dist = reinterpret_cast<int32_t*>(ws + L.dist);
    a.vis = reinterpret_cast<uint32_t*>(ws + L.vis);
    a.sig = reinterpret_cast<uint32_t*>(ws + L.sig);
    a.part = reinterpret_cast<double*>(ws + L.part);
    a.arrived = reinterpret_cast<int32_t*>(ws + L.arrived);
    a.st = reinterpret_cast<BcPullState*>(ws + L.st);
    a.perm = g->d.perm;
    a.bc = bc;
    uint32_t* buf[2] = {reinterpret_cast<uint32_t*>(ws + L.f0), reinterpret_cast<uint32_t*>(ws + L.f1)};
    BcUnit* units[2] = {reinterpret_cast<BcUnit*>(ws + L.units0), reinterpret_cast<BcUnit*>(ws + L.units1)};
    const int32_t vb = std::max(1, std::min(ceil_div(n, kBlock), 4096));
    const int32_t grid = std::max(1, std::min(ceil_div(n, kBcRows * kBcWaves), 6 * g->num_cu));
    a.share = 8;
    while (a.share > 1 && (int64_t)ceil_div(n, kWave) * a.share > 2 * (int64_t)grid * kBcWaves) a.share /= 2;
    hipLaunchKernelGGL(k_bc_zero, dim3(vb), dim3(kBlock), 0, st, n, bc);
    BcPullState zero{};
    PP_HIP(hipMemcpyAsync(a.st, &zero, sizeof(zero), hipMemcpyHostToDevice, st));
    for (int side = 0; side < (symmetric ? 1 : 2); ++side)
        hipLaunchKernelGGL(k_bc_units, dim3(ceil_div(n, kBlock)), dim3(kBlock), 0, st, n,
                           side ? g->d.csr_off : g->d.csc_off, units[side], a.arrived, &a.st->units[side],
                           &a.st->parts[side]);
    PP_LAUNCH_CHECK("k_bc_units");
    // forward kernels per launch batch, then one more than the last depth seen
    // (an empty level is about 3 us, a look at the state 20)
    int32_t batch = 8;
    for (int32_t k0 = 0; k0 < num_sources; k0 += KP) {
        const int32_t cnt = std::min(KP, num_sources - k0);
        BcSources src{};
        for (int32_t i = 0; i < cnt; ++i) src.s[i] = sources[k0 + i];
        a.all = cnt == 32 ? 0xFFFFFFFFu : (1u << cnt) - 1u;
        a.off = g->d.csc_off;
        a.idx = g->d.csc_idx;
        a.units = units[0];
        a.side = 0;
        a.fn = buf[0];
        hipLaunchKernelGGL(k_bc_begin<KP>, dim3(vb), dim3(kBlock), 0, st, a, src, cnt, g->d.iperm);
        int32_t l = 0;
        BcPullState hs{};
        for (;;) {
            for (int32_t i = 0; i < batch; ++i, ++l) {
                a.fm = buf[l & 1];
                a.fn = buf[(l + 1) & 1];
                hipLaunchKernelGGL((k_bc_level<KP, true>), dim3(grid), dim3(kBlock), 0, st, a, l);
            }
            PP_LAUNCH_CHECK("k_bc_level");
            PP_HIP(hipMemcpyAsync(&hs, a.st, sizeof(hs), hipMemcpyDeviceToHost, st));
            PP_HIP(hipStreamSynchronize(st));
            if (!hs.any[l % 3] || l > n) break;
            batch = std::min(batch * 2, 64);
        }
        batch = std::max(2, hs.depth + 1);
        // the deepest level has no successors; the sources' own (level 0) do
        // not count
        a.off = g->d.csr_off;
        a.idx = g->d.csr_idx;
        a.units = units[symmetric ? 0 : 1];
        a.side = symmetric ? 0 : 1;
        for (l = hs.depth - 1; l > 0; --l) {
            a.fm = l == hs.depth - 1 ? nullptr : buf[(l + 1) & 1];
            a.fn = buf[l & 1];
            hipLaunchKernelGGL((k_bc_level<KP, false>), dim3(grid), dim3(kBlock), 0, st, a, l);
        }
        PP_LAUNCH_CHECK("k_bc_level");
    }
    return PP_OK;
}

}  // namespace pp

using namespace pp;

PP_EXPORT size_t pp_bc_workspace_bytes(pp_graph g) { return g ? kBcStates + kBcBatch * bc_layout(g->d.n).slab : 0; }

PP_EXPORT pp_status pp_bc_run(pp_graph g, pp_dir fwd_dir, pp_dir bwd_dir, int32_t num_sources,
                              const int32_t* sources, double* bc, void* ws, size_t ws_bytes, void* stream) {
    clear_error();
    if (!g) return set_error(PP_E_NULL, "graph handle is NULL");
    if (!bc || !ws || (num_sources > 0 && !sources)) return set_error(PP_E_NULL, "bc, ws and sources are required");
    if ((fwd_dir != PP_PUSH && fwd_dir != PP_PULL) || (bwd_dir != PP_PUSH && bwd_dir != PP_PULL))
        return set_error(PP_E_RANGE, "directions must be PP_PUSH or PP_PULL");
    if (num_sources < 0) return set_error(PP_E_RANGE, "num_sources must be >= 0");
    const int32_t n = g->d.n;
    for (int32_t k = 0; k < num_sources; ++k)
        if (sources[k] < 0 || sources[k] >= n) return set_error(PP_E_RANGE, "source out of range");
    const BcLayout L = bc_layout(n);
    if (ws_bytes < kBcStates + L.slab) return set_error(PP_E_WORKSPACE, "BC workspace too small");
    if (reinterpret_cast<uintptr_t>(ws) % 256 != 0) return set_error(PP_E_RANGE, "ws must be 256-byte aligned");
    // as many sources at once as the workspace holds, at most kBcBatch
    const int32_t per_batch = (int32_t)std::min<size_t>(kBcBatch, (ws_bytes - kBcStates) / L.slab);
    char* w = static_cast<char*>(ws);
    // Shared levels cost a launch about 0.5 us more of load latency than the
    // per-source ones, which tells where the levels are many and have little in
    // them: low degrees on few vertices and sources (a path of 3,000 vertices, 1
    // and 32 sources: 13.6 and 27.6 ms per source, 17.4 and 37.6 shared; a 100^2
    // grid 1.6 against 1.9 with one source, 3.2 against 3.1 with 32; a 300^2 grid
    // 7.9 against 9.0 with one, 15.6 against 10.5 with 4, 60 against 15 with 32).
    const int32_t want = std::min(per_batch, num_sources);
    if (fwd_dir == PP_PULL && bwd_dir == PP_PULL && num_sources > 0 &&
        (g->d.nnz >= 8 * (int64_t)n || (int64_t)n * want >= 300000)) {
        const int kp = want > 16 ? 32 : want > 8 ? 16 : want > 4 ? 8 : 4;
        const bool symmetric = g->d.csr_off == g->d.csc_off && g->d.csr_idx == g->d.csc_idx;
        const BcPullLayout P = bc_pull_layout(n, g->d.nnz, kp, symmetric);
        if (P.total <= ws_bytes) {
            hipStream_t ps = static_cast<hipStream_t>(stream);
            switch (kp) {
                case 32: return bc_pull_run<32>(g, P, num_sources, sources, bc, w, ps);
                case 16: return bc_pull_run<16>(g, P, num_sources, sources, bc, w, ps);
                case 8: return bc_pull_run<8>(g, P, num_sources, sources, bc, w, ps);
                default: return bc_pull_run<4>(g, P, num_sources, sources, bc, w, ps);
            }
        }
    }
    char* slab0 = w + kBcStates;
    BcArgs a;
    a.n = n;
    a.hot = std::min(n, kBcHot);
    a.out_off = g->d.csr_off;
    a.out_idx = g->d.csr_idx;
    a.in_off = g->d.csc_off;
    a.in_idx = g->d.csc_idx;
    a.perm = g->d.perm;
    a.iperm = g->d.iperm;
    a.dist = reinterpret_cast<int32_t*>(slab0 + L.dist);
    a.sigma = reinterpret_cast<double*>(slab0 + L.sigma);
    a.delta = reinterpret_cast<double*>(slab0 + L.delta);
    a.order = reinterpret_cast<int32_t*>(slab0 + L.order);
    a.cnt = reinterpret_cast<int32_t*>(slab0 + L.cnt);
    a.lvl_off = reinterpret_cast<int32_t*>(slab0 + L.lvl_off);
    a.st = reinterpret_cast<BcState*>(w);
    a.stride = L.slab;
    a.bc = bc;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const int32_t vb = std::max(1, std::min(ceil_div(n, kBlock), 4096));
    // per source: every pushing workgroup zeroes and flushes its hot
    // accumulators, so a few per compute unit, over all sources of a batch (64 at
    // R-MAT 16: 5.1 ms at 2 a compute unit and source, 4.7 at 8 and 4.5 at 16 a
    // compute unit, 5.3 at 4); the pulling kernels sweep vertex or level lists
    // grid-stride
    const int32_t share = 16 * g->num_cu / std::max(1, std::min(per_batch, num_sources));
    const int32_t pb = std::max(1, std::min(std::min(ceil_div(n, kBlock), 2 * g->num_cu), share));
    const int32_t fx = (fwd_dir == PP_PUSH) ? pb : vb;
    const int32_t bx = (bwd_dir == PP_PUSH) ? pb : std::min(vb, 2 * g->num_cu);
    hipLaunchKernelGGL(k_bc_zero, dim3(vb), dim3(kBlock), 0, st, n, bc);
    PP_LAUNCH_CHECK("k_bc_zero");
    std::vector<BcState> hs(per_batch);
    int32_t batch = 4;  // forward kernels per launch batch: one more than the last depth seen
    for (int32_t k0 = 0; k0 < num_sources; k0 += per_batch) {
        const int32_t cnt = std::min(per_batch, num_sources - k0);
        BcSources src{};
        for (int32_t i = 0; i < cnt; ++i) src.s[i] = sources[k0 + i];
        hipLaunchKernelGGL(k_bc_init, dim3(vb, cnt), dim3(kBlock), 0, st, a, src);
        // forward levels in batches; a source past its last level returns at once
        int32_t launched = 0, depth = 0;
        for (;;) {
            for (int32_t i = 0; i < batch; ++i) {
                if (fwd_dir == PP_PUSH) hipLaunchKernelGGL(k_bc_fwd_push, dim3(fx, cnt), dim3(kBlock), 0, st, a);
                else hipLaunchKernelGGL(k_bc_fwd_pull, dim3(fx, cnt), dim3(kBlock), 0, st, a);
            }
            PP_LAUNCH_CHECK("k_bc_fwd");
            launched += batch;
            PP_HIP(hipMemcpyAsync(hs.data(), a.st, sizeof(BcState) * cnt, hipMemcpyDeviceToHost, st));
            PP_HIP(hipStreamSynchronize(st));
            bool all = true;
            depth = 0;
            for (int32_t i = 0; i < cnt; ++i) {
                all = all && hs[i].done;
                depth = std::max(depth, hs[i].depth);
            }
            if (all || launched > n) break;
            batch = std::min(batch * 2, 64);
        }
        batch = std::max(2, depth + 1);
        // backward levels D-2 .. 0 of each source, its state counting down
        for (int32_t l = depth - 2; l >= 0; --l) {
            if (bwd_dir == PP_PUSH) hipLaunchKernelGGL(k_bc_bwd_push, dim3(bx, cnt), dim3(kBlock), 0, st, a);
            else hipLaunchKernelGGL(k_bc_bwd_pull, dim3(bx, cnt), dim3(kBlock), 0, st, a);
        }
        hipLaunchKernelGGL(k_bc_acc, dim3(vb), dim3(kBlock), 0, st, a, src, cnt);
        PP_LAUNCH_CHECK("k_bc_bwd");
    }
    return PP_OK;
}
