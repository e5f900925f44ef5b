// The routed PageRank sweep: y[u] = teleport + sum of the contributions that
// reach u, in two passes that touch memory in order only.
//
// A gather (or a scatter) of one 4-byte value per edge over a vector larger
// than a compute unit's LDS runs at the chip's random-access rate (81 G/s
// over 17 MB, 121 G/s over 8 MB), ten times below what the bytes alone would
// allow.  Here the edges are routed instead:
//   1. k_route_send: sources are taken slice by slice (kRouteWidth consecutive
//      ids, staged in LDS), and the value of every edge that leaves the slice
//      is written to the mailbox of its target block -- one in-order stream of
//      16-bit source offsets in, one in-order stream of values out;
//   2. k_route_sum: a workgroup owns a block of consecutive in-edge slots,
//      reads its mailbox (one run per slice), places every value at its slot
//      in LDS (16-bit positions) and sums each row from there.
// 12 bytes an edge instead of a 64-byte line (2 + 4 out, 4 + 2 in), and the
// values of up to 64M edges stay in the memory-side cache between the passes.
// ER n = 3,000,017 (48M edges), a step: 57 + 72 us (5.0 and 4.5 TB/s), against
// 583 us gathered; R-MAT 20 pushed: 43 + 58 us, against 258 us of LDS atomics
// and binned updates.
// No atomics; a row is summed in a fixed order of its stored slots, so the
// result is bit-reproducible.
//
// Seen from the sources this is the pushing sweep with buffered remote updates
// (Sec. 5 Partition-Awareness: the block is the owner, nothing is shared but
// its mailbox); seen from the targets it is the pulling sweep with its gathers
// moved ahead.  Both forms use it where it pays (route_for).
#include <hip/hip_runtime.h>

#include <vector>

#include "pp_common.h"

namespace pp {

// ------------------------------------------------------------------ plan
// Slot range and rows of a block.
__global__ void k_route_blocks(int32_t blocks, int64_t nnz, const int32_t* __restrict__ off,
                               const int32_t* __restrict__ row, RouteBlock* __restrict__ blk) {
    const int32_t k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= blocks) return;
    // a cut falls at the end of the row it lands in, or inside a long row
    auto cut = [&](int64_t t) -> int32_t {
        if (t >= nnz) return (int32_t)nnz;
        const int32_t r = row[t];
        const int32_t b = off[r], e = off[r + 1];
        return (b == t || e - b > kRouteSlack) ? (int32_t)t : e;
    };
    RouteBlock o;
    o.p0 = cut((int64_t)k * kRouteEdges);
    o.p1 = cut((int64_t)(k + 1) * kRouteEdges);
    o.r0 = o.p0 < o.p1 ? row[o.p0] : 0;
    o.r1 = o.p0 < o.p1 ? row[o.p1 - 1] : 0;  // an empty last block: row 0 owns no slot of it
    blk[k] = o;
}

// Edges of every (slice, block) run, slice-major.
__global__ __launch_bounds__(256) void k_route_count(int32_t S, int32_t B, const RouteBlock* __restrict__ blk,
                                                     const int32_t* __restrict__ idx, int32_t* __restrict__ cnt) {
    __shared__ int32_t h[kRouteMaxSlices];
    for (int32_t s = threadIdx.x; s < S; s += blockDim.x) h[s] = 0;
    __syncthreads();
    const RouteBlock k = blk[blockIdx.x];
    for (int32_t j = k.p0 + threadIdx.x; j < k.p1; j += blockDim.x) atomicAdd(&h[idx[j] >> kRouteShift], 1);
    __syncthreads();
    // runs start at multiples of four entries (wide loads)
    for (int32_t s = threadIdx.x; s < S; s += blockDim.x) cnt[(size_t)s * B + blockIdx.x] = (h[s] + 3) & ~3;
}

// Run starts, block-major, and how many runs are not empty.
__global__ void k_route_runs(int32_t S, int32_t B, const int32_t* __restrict__ start, int32_t* __restrict__ run,
                             int32_t* __restrict__ used) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    bool some = false;
    if (t < (int64_t)S * (B + 1)) {
        const int32_t b = (int32_t)(t / S), s = (int32_t)(t % S);
        const size_t at = (size_t)s * B + b;  // row B: the end of the slice
        run[t] = start[at];
        some = b < B && start[at + 1] > start[at];
    }
    const uint64_t m = __ballot(some);
    if (m && (threadIdx.x & (kWave - 1)) == 0) atomicAdd(used, __popcll(m));
}

// Source offset and slot position of every edge, in run order (the order
// inside a run does not reach the sums: values are placed by slot).
__global__ __launch_bounds__(256) void k_route_fill(int32_t S, const RouteBlock* __restrict__ blk,
                                                    const int32_t* __restrict__ idx, const int32_t* __restrict__ run,
                                                    uint16_t* __restrict__ src, uint16_t* __restrict__ pos) {
    __shared__ int32_t cur[kRouteMaxSlices];
    for (int32_t s = threadIdx.x; s < S; s += blockDim.x) cur[s] = run[(size_t)blockIdx.x * S + s];
    __syncthreads();
    const RouteBlock k = blk[blockIdx.x];
    for (int32_t j = k.p0 + threadIdx.x; j < k.p1; j += blockDim.x) {
        const int32_t v = idx[j];
        const int32_t e = atomicAdd(&cur[v >> kRouteShift], 1);
        src[e] = (uint16_t)(v & (kRouteWidth - 1));
        pos[e] = (uint16_t)(j - k.p0);
    }
    __syncthreads();
    for (int32_t s = threadIdx.x; s < S; s += blockDim.x)
        for (int32_t e = cur[s]; e < run[(size_t)(blockIdx.x + 1) * S + s]; ++e) {
            src[e] = 0;
            pos[e] = (uint16_t)kRouteSlots;  // a padding entry's value goes to a spare place
        }
}

// ------------------------------------------------------------------ sweep
struct RouteArgs {
    int32_t n, S, B;
    int32_t entries;          // of the stream, paddings included
    int32_t quota;            // entries of one sending workgroup (a multiple of 4)
    const uint16_t* src;
    const uint16_t* pos;
    float* val;
    const int32_t* run;       // [(B + 1) * S] run starts, block-major
    const RouteBlock* blk;
    float* head;              // [B] sum of a row that began in an earlier block
    float* tail;              // [B] sum of a row that goes on in the next block
    const float* c;
    const int32_t* off;       // CSC offsets
    const float* wt;          // weights in CSC slot order (weighted only)
    const float* inv_s;
    const int32_t* perm;
    float* c_next;
    float* y;
    int64_t y_stride;
    float base, tele, f;
    int32_t tele_v;
};

// What the owner of a row needs besides its sum, loaded ahead of it.
struct RouteRow {
    int32_t ob, oe;  // slots
    float inv_s;
};
__device__ __forceinline__ RouteRow route_load(const RouteArgs& a, int32_t u) {
    RouteRow w;
    w.ob = a.off[u];
    w.oe = a.off[u + 1];
    w.inv_s = a.c_next ? a.inv_s[u] : 0.f;
    return w;
}

__device__ __forceinline__ void route_finish(const RouteArgs& a, int32_t u, float inv_s, float acc) {
    const float yv = a.base + ((u == a.tele_v) ? a.tele : 0.f) + acc;
    if (a.y) a.y[(int64_t)user_id(a.perm, u) * a.y_stride] = yv;
    if (a.c_next) a.c_next[u] = a.f * yv * inv_s;
}

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

// Workgroup w sends entries [w * quota, (w + 1) * quota) of the slice-major
// stream, staging every slice it meets.  A lane takes four entries at a time:
// an 8-byte load, four LDS reads, a 16-byte store.
__global__ __launch_bounds__(1024) void k_route_send(RouteArgs a) {
    extern __shared__ float s_c[];  // kRouteWidth contributions
    const int32_t e0 = (int32_t)min((int64_t)blockIdx.x * a.quota, (int64_t)a.entries);
    const int32_t e1 = (int32_t)min((int64_t)e0 + a.quota, (int64_t)a.entries);
    if (e0 >= e1) return;
    const int32_t* start = a.run;                      // of every slice
    const int32_t* stop = a.run + (size_t)a.B * a.S;
    int32_t lo = 0, hi = a.S - 1;  // the slice that holds e0: the first with stop > e0
    while (lo < hi) {
        const int32_t mid = (lo + hi) >> 1;
        if (stop[mid] > e0) hi = mid;
        else lo = mid + 1;
    }
    for (int32_t s = lo; s < a.S; ++s) {
        const int32_t b = max(start[s], e0), e = min(stop[s], e1);
        if (start[s] >= e1) break;
        if (b >= e) continue;
        const int32_t v0 = s << kRouteShift, count = min(kRouteWidth, a.n - v0);
        __syncthreads();  // the previous slice is read
        for (int32_t i = threadIdx.x * 4; i + 3 < count; i += blockDim.x * 4)
            *reinterpret_cast<float4*>(s_c + i) = *reinterpret_cast<const float4*>(a.c + v0 + i);
        for (int32_t i = (count & ~3) + threadIdx.x; i < count; i += blockDim.x) s_c[i] = a.c[v0 + i];
        __syncthreads();
        // [b, e) starts and ends at multiples of four entries
        constexpr int U = 4;
        const int32_t step = blockDim.x * 4;
        for (int32_t q0 = b + threadIdx.x * 4; q0 < e; q0 += U * step) {
            u32x2 w[U];
#pragma unroll
            for (int k = 0; k < U; ++k)
                w[k] = __builtin_nontemporal_load(reinterpret_cast<const u32x2*>(a.src + min(q0 + k * step, e - 4)));
#pragma unroll
            for (int k = 0; k < U; ++k) {
                const int32_t q = q0 + k * step;
                const float4 v = make_float4(s_c[w[k].x & 0xFFFFu], s_c[w[k].x >> 16], s_c[w[k].y & 0xFFFFu],
                                             s_c[w[k].y >> 16]);
                if (q < e) *reinterpret_cast<float4*>(a.val + q) = v;
            }
        }
    }
}

// Sum of the placed slots [b, e) (positions in the block) by G lanes.
template <bool W>
__device__ __forceinline__ float route_row(const RouteArgs& a, const float* s_v, int32_t p0, int32_t b, int32_t e,
                                           int gl, int G) {
    float q[4] = {0.f, 0.f, 0.f, 0.f};  // four sums: a hub's slots add up in short chains
    for (int32_t i0 = b + gl; i0 < e; i0 += 4 * G) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int32_t i = min(i0 + k * G, e - 1);
            const float v = W ? s_v[i] * a.wt[p0 + i] : s_v[i];
            q[k] += (i0 + k * G < e) ? v : 0.f;
        }
    }
    float acc = (q[0] + q[1]) + (q[2] + q[3]);
    for (int s = G >> 1; s > 0; s >>= 1) acc += __shfl_xor(acc, s);
    return acc;
}

// A row's sum in block b: the whole row, its end or its beginning (lane 0).
__device__ __forceinline__ void route_put(const RouteArgs& a, const RouteBlock& k, int32_t b, int32_t r,
                                          const RouteRow& w, float acc, int lane) {
    if (lane != 0) return;
    if (w.ob < k.p0) a.head[b] = acc;
    else if (w.oe > k.p1) a.tail[b] = acc;
    else route_finish(a, r, w.inv_s, acc);
}

// One block: mailbox to LDS, then the rows.  The runs are cut into pieces of
// kRoutePiece entries (a skewed graph's first slices send half of a block in
// one run), 16 lanes a piece.  Rows take G lanes, G by the block's row
// count; rows of more than 32 G slots are left to
// whole wavefronts.  Blocks past B finish the rows without in-edges.
constexpr int kRouteLanes = 16;
constexpr int kRoutePiece = kRouteLanes * 4;
template <bool W>
__global__ __launch_bounds__(1024) void k_route_sum(RouteArgs a) {
    __shared__ float s_v[kRouteSlots + 4];  // and the place of the padding entries
    __shared__ int2 s_piece[kRouteMaxSlices + kRouteSlots / kRoutePiece];  // (first entry, entries)
    __shared__ int32_t s_count[2];  // pieces, long rows
    int32_t* s_long = reinterpret_cast<int32_t*>(s_piece);  // the pieces are done with by then
    static_assert(sizeof(s_piece) >= (kRouteSlots / 33 + 1) * 4, "long rows of a block");
    if ((int32_t)blockIdx.x >= a.B) {
        const int32_t u = ((int32_t)blockIdx.x - a.B) * (int32_t)blockDim.x + (int32_t)threadIdx.x;
        if (u < a.n) {
            const RouteRow w = route_load(a, u);
            if (w.ob == w.oe) route_finish(a, u, w.inv_s, 0.f);
        }
        return;
    }
    const int32_t b = blockIdx.x;
    const RouteBlock k = uniform_load(a.blk, b);
    const int lane = threadIdx.x & (kWave - 1);
    // lanes a row: as many as leave the workgroup one pass over the rows or so;
    // the first pass's bounds load beside the run table
    const int32_t rows = k.r1 - k.r0 + 1;
    int G = 1;
    while (G < kWave && rows * (2 * G) <= (int32_t)blockDim.x * 3 / 2) G <<= 1;
    const int32_t row0 = k.r0 + (int32_t)threadIdx.x / G, rstep = (int32_t)blockDim.x / G;
    RouteRow row = route_load(a, min(row0, k.r1));
    if (threadIdx.x < 2) s_count[threadIdx.x] = 0;
    __syncthreads();
    const int32_t* r0 = a.run + (size_t)b * a.S;
    for (int32_t s0 = threadIdx.x - lane; s0 < a.S; s0 += blockDim.x) {
        const int32_t s = s0 + lane;
        const int32_t lo = s < a.S ? r0[s] : 0, hi = s < a.S ? r0[s + a.S] : 0;
        const int32_t np = (hi - lo + kRoutePiece - 1) / kRoutePiece;
        int32_t sum = np;
#pragma unroll
        for (int d = 1; d < kWave; d <<= 1) {
            const int32_t o = __shfl_up(sum, d);
            if (lane >= d) sum += o;
        }
        int32_t at = 0;
        if (lane == kWave - 1) at = atomicAdd(&s_count[0], sum);
        at = __shfl(at, kWave - 1) + sum - np;
        for (int32_t i = 0; i < np; ++i)
            s_piece[at + i] = make_int2(lo + i * kRoutePiece, min(kRoutePiece, hi - lo - i * kRoutePiece));
    }
    __syncthreads();
    const int gl = threadIdx.x & (kRouteLanes - 1);
    const int32_t pieces = s_count[0];
    constexpr int U = 2;
    const int32_t ngrp = blockDim.x / kRouteLanes;
    for (int32_t i0 = threadIdx.x / kRouteLanes; i0 < pieces; i0 += U * ngrp) {
        float4 v[U];
        u32x2 p[U];
        bool live[U];
#pragma unroll
        for (int q = 0; q < U; ++q) {
            const int2 pc = s_piece[min(i0 + q * ngrp, pieces - 1)];
            live[q] = i0 + q * ngrp < pieces && 4 * gl < pc.y;
            const int32_t e = pc.x + min(4 * gl, pc.y - 4);
            v[q] = *reinterpret_cast<const float4*>(a.val + e);
            p[q] = __builtin_nontemporal_load(reinterpret_cast<const u32x2*>(a.pos + e));
        }
#pragma unroll
        for (int q = 0; q < U; ++q)
            if (live[q]) {
                s_v[p[q].x & 0xFFFFu] = v[q].x;
                s_v[p[q].x >> 16] = v[q].y;
                s_v[p[q].y & 0xFFFFu] = v[q].z;
                s_v[p[q].y >> 16] = v[q].w;
            }
    }
    __syncthreads();
    const int32_t gr = threadIdx.x & (G - 1);
    for (int32_t r = row0; r <= k.r1; r += rstep) {
        const RouteRow w = row;
        row = route_load(a, min(r + rstep, k.r1));
        const int32_t rb = max(w.ob, k.p0), re = min(w.oe, k.p1);
        if (re <= rb) continue;
        if (G < kWave && re - rb > 32 * G) {
            if (gr == 0) s_long[atomicAdd(&s_count[1], 1)] = r;
            continue;
        }
        route_put(a, k, b, r, w, route_row<W>(a, s_v, k.p0, rb - k.p0, re - k.p0, gr, G), gr);
    }
    __syncthreads();
    for (int32_t i = threadIdx.x / kWave; i < s_count[1]; i += blockDim.x / kWave) {
        const int32_t r = s_long[i];
        const RouteRow w = route_load(a, r);
        route_put(a, k, b, r, w,
                  route_row<W>(a, s_v, k.p0, max(w.ob, k.p0) - k.p0, min(w.oe, k.p1) - k.p0, lane, kWave), lane);
    }
}

// Rows that cross blocks: the pieces in slot order.
__global__ void k_route_fix(RouteArgs a) {
    const int32_t b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b < 1 || b >= a.B) return;
    const RouteBlock k = a.blk[b];
    if (k.p0 >= k.p1) return;
    const int32_t ob = a.off[k.r0], oe = a.off[k.r0 + 1];
    if (ob >= k.p0 || ob < a.blk[b - 1].p0) return;  // not the row's second block
    float acc = a.tail[b - 1];
    for (int32_t q = b; q < a.B && a.blk[q].p0 < oe; ++q) acc += a.head[q];
    route_finish(a, k.r0, a.c_next ? a.inv_s[k.r0] : 0.f, acc);
}

// ------------------------------------------------------------------ host side
// Graphs the routed sweep is planned for: edges enough that its two launches
// pay, slices that fit the planning kernels' counters.
bool route_possible(int32_t n, int64_t nnz) {
    return n >= kRouteMinN && nnz <= INT32_MAX / 2 && ceil_div(n, kRouteWidth) <= kRouteMaxSlices && nnz >= kRouteMinEdges;
}

// Entries of the stream, at most: up to three paddings a run, in no more runs
// than edges.
static size_t route_slots(int32_t n, int64_t nnz) {
    const int64_t cells = (int64_t)ceil_div(n, kRouteWidth) * ceil_div(nnz, kRouteEdges);
    return align_up((size_t)(nnz + 3 * std::min(cells, nnz)), 8);
}

size_t route_edge_bytes(int32_t n, int64_t nnz) { return route_slots(n, nnz) * 8; }

size_t route_table_bytes(int32_t n, int64_t nnz) {
    const size_t S = ceil_div(n, kRouteWidth), B = ceil_div(nnz, kRouteEdges);
    return align_up((B + 1) * S * 4, 256) + align_up(B * sizeof(RouteBlock), 256) + 2 * align_up(B * 4, 256);
}

// Whether the pulling form is routed as well.  The plain pull stages the first
// pull_hot contributions in LDS and gathers the rest from cache, so it loses
// where most gathers miss the stage and go all over a vector that is not small
// (a step, plain -> routed): ER n = 120,001 21.4 -> 20.4 us, 200,001 27.5 ->
// 24.7, 1M 126 -> 53, 2M 316 -> 90 (missed: 73-98% of the gathers).  On R-MAT
// 17-20 6-32% miss and the plain pull stays ahead (20: 82 against 107 us); past
// 2^20 vertices the vector outgrows an XCD's 4 MB L2 and 40% are enough (R-MAT
// 21: 212 -> 195).  A grid's gathers miss the stage but sit side by side (its
// blocks meet few of the slices): plain 8.7, routed 19.8 us at n = 100,000.
static bool route_pull_pays(pp_graph g, int64_t entries, int64_t staged, int64_t used, int64_t cells) {
    const int64_t missed = entries - staged;
    if (g->d.n < 4 * kRouteWidth || used * 4 < cells * 3) return false;
    return missed * 8 >= entries * (g->d.n > (1 << 20) ? 3 : 5);
}

// Plans the routed sweep over the registered in-adjacency.  `edges`:
// route_edge_bytes, `tables`: route_table_bytes, both in the graph workspace.
pp_status build_route(pp_graph g, void* edges, void* tables, hipStream_t st) {
    g->route = RoutePlan{};
    GraphDev& d = g->d;
    if (!route_possible(d.n, d.nnz)) return PP_OK;
    if ((int32_t)(kRouteWidth * sizeof(float)) > g->max_lds) return PP_OK;
    const int32_t S = ceil_div(d.n, kRouteWidth), B = ceil_div(d.nnz, kRouteEdges);
    char* w = static_cast<char*>(tables);
    d.rt_run = reinterpret_cast<int32_t*>(w);
    w += align_up((size_t)(B + 1) * S * 4, 256);
    d.rt_blk = reinterpret_cast<RouteBlock*>(w);
    w += align_up((size_t)B * sizeof(RouteBlock), 256);
    d.rt_head = reinterpret_cast<float*>(w);
    w += align_up((size_t)B * 4, 256);
    d.rt_tail = reinterpret_cast<float*>(w);
    d.rt_val = static_cast<float*>(edges);
    d.rt_src = reinterpret_cast<uint16_t*>(d.rt_val + route_slots(d.n, d.nnz));
    d.rt_pos = d.rt_src + route_slots(d.n, d.nnz);
    // counts and their scan live in the value stream until the first sweep
    const int64_t cells = (int64_t)S * B;
    int32_t* cnt = reinterpret_cast<int32_t*>(d.rt_val);
    int32_t* start = cnt + cells;
    int32_t* sums = start + cells + 1;
    if (2 * cells + 1 + ceil_div(cells, 1024) + 1 > d.nnz) return PP_OK;
    hipLaunchKernelGGL(k_route_blocks, dim3(ceil_div(B, 256)), dim3(256), 0, st, B, d.nnz, d.csc_off, d.csc_row,
                       d.rt_blk);
    hipLaunchKernelGGL(k_route_count, dim3(B), dim3(256), 0, st, S, B, (const RouteBlock*)d.rt_blk, d.csc_idx, cnt);
    PP_LAUNCH_CHECK("route count");
    pp_status s = exclusive_scan((int32_t)cells, cnt, start, sums, d.err + 40, st);
    if (s != PP_OK) return s;
    hipLaunchKernelGGL(k_route_runs, dim3(ceil_div((int64_t)S * (B + 1), 256)), dim3(256), 0, st, S, B,
                       (const int32_t*)start, d.rt_run, d.err + 41);
    PP_LAUNCH_CHECK("route runs");
    int32_t h[3] = {0, 0, 0};  // entries, runs in use, entries whose source a plain pull stages
    const int32_t staged = std::min(std::max(g->tune.pull_hot, 0) >> kRouteShift, S);
    PP_HIP(hipMemcpyAsync(h, d.err + 40, 8, hipMemcpyDeviceToHost, st));
    PP_HIP(hipMemcpyAsync(h + 2, start + (int64_t)staged * B, 4, hipMemcpyDeviceToHost, st));
    PP_HIP(hipStreamSynchronize(st));
    if (h[0] < d.nnz || (size_t)h[0] > route_slots(d.n, d.nnz)) return set_error(PP_E_GRAPH, "routed sweep: run table");
    hipLaunchKernelGGL(k_route_fill, dim3(B), dim3(256), 0, st, S, (const RouteBlock*)d.rt_blk, d.csc_idx,
                       (const int32_t*)d.rt_run, d.rt_src, d.rt_pos);
    PP_LAUNCH_CHECK("route fill");
    g->route.entries = h[0];
    g->route.slices = S;
    g->route.blocks = B;
    g->route.split = g->max_in_deg > kRouteSlack;
    g->route.pull = route_pull_pays(g, h[0], h[2], h[1], cells);
    return PP_OK;
}

// Which sweeps take the routed path: pulls without a tiled plan where it pays,
// pushes whose remote updates are buffered (pp_set_push_bins).  No plan is made
// where the in-adjacency is not the transpose.
bool route_for(pp_graph g, pp_dir dir) {
    if (g->route.blocks == 0) return false;
    return dir == PP_PULL ? (g->route.pull && g->slices.rows == 0) : (g->tune.push_bins && g->tune.hot > 0 && g->transposed);
}

// One routed sweep: y and / or the next contributions from c.
pp_status launch_route(pp_graph g, const float* c, float* c_next, float* y, float f, hipStream_t st,
                       const Teleport* tpp) {
    const Teleport tp = tpp ? *tpp : uniform_teleport(g->d.n, f);
    const GraphDev& d = g->d;
    RouteArgs a{};
    a.n = d.n;
    a.S = g->route.slices;
    a.B = g->route.blocks;
    a.entries = g->route.entries;
    a.quota = (ceil_div(a.entries, g->num_cu) + 3) & ~3;
    a.src = d.rt_src;
    a.pos = d.rt_pos;
    a.val = d.rt_val;
    a.run = d.rt_run;
    a.blk = d.rt_blk;
    a.head = d.rt_head;
    a.tail = d.rt_tail;
    a.c = c;
    a.off = d.csc_off;
    a.wt = d.csc_w;
    a.inv_s = d.inv_s;
    a.perm = d.perm;
    a.c_next = c_next;
    a.y = y;
    a.y_stride = tp.y_stride;
    a.base = tp.base;
    a.tele_v = tp.vertex;
    a.tele = tp.extra;
    a.f = f;
    const size_t lds = (size_t)kRouteWidth * sizeof(float);
    allow_dynamic_lds(reinterpret_cast<const void*>(&k_route_send), lds);
    hipLaunchKernelGGL(k_route_send, dim3(ceil_div(a.entries, a.quota)), dim3(1024), lds, st, a);
    const int32_t tail = g->empty_in > 0 ? ceil_div(d.n, 1024) : 0;
    if (g->weighted) hipLaunchKernelGGL((k_route_sum<true>), dim3(a.B + tail), dim3(1024), 0, st, a);
    else hipLaunchKernelGGL((k_route_sum<false>), dim3(a.B + tail), dim3(1024), 0, st, a);
    if (g->route.split) hipLaunchKernelGGL(k_route_fix, dim3(ceil_div(a.B, 64)), dim3(64), 0, st, a);
    PP_LAUNCH_CHECK("k_route_send");
    return PP_OK;
}

}  // namespace pp
