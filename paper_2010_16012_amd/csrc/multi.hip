// Many small graphs in one call: PageRank (push or pull) and BFS for every
// graph of a concatenated arena, one workgroup per graph.
//
// Parallelism beyond one graph (the paper's sweeps are per graph; Sec. 4
// assumes up to one processor per vertex): a graph of at most kMultiMaxN
// vertices keeps its whole per-vertex state in the LDS of one compute unit,
// so the pull gathers and the push updates are LDS operations (ds_read /
// ds_add_f32) and the barrier between two sweeps is a workgroup barrier --
// no grid-wide synchronisation, no spin waits.  Workgroups take graphs
// largest first (longest-processing-time order) so the big graphs start
// first and small ones fill in.
//
// One compute unit sweeps about 3.5 edges a nanosecond, so a batch with large
// graphs waited for the largest alone (a scale-14 R-MAT graph: 134 us a sweep,
// 2.7 of the 3.1 ms of a 128-graph batch, most of the chip idle).  Where a graph
// has more than kStepEdges edges and is more than its share (steps_pay) the
// PageRank steps therefore run as one launch each (k_multi_step), the rows of all
// graphs shared among one workgroup per compute unit: 40 us a step there, 1.07 ms
// in all.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <mutex>
#include <numeric>
#include <string>
#include <type_traits>
#include <vector>

#include "pp_common.h"

namespace pp {

constexpr int kMultiBlock = 1024;
constexpr int kMultiGroup = 4;  // lanes per row
constexpr int kMultiU = 8;      // index loads in flight per lane
constexpr int kMultiPullU = 8;  // slots per lane and round of a pull row
constexpr int32_t kMultiMaxN = 16384;
// PageRank rows at least `big` long (tuned; 512 by default) get a whole
// wavefront each (up to kMultiBigCap of them per graph); a small group per
// row would leave the wavefront holding the hubs running long after the
// others.
constexpr int32_t kMultiBigCap = 512;
// Rows of `mid`..`big`-1 edges (64 by default) go to groups of ML lanes
// (tuned; 16 by default), up to kMultiMidCap of them per graph: in a small
// group such a row takes several rounds while the wavefront's other rows
// wait.  The short pull rows take PG lanes each (tuned; 2 by default; the
// push and BFS use kMultiGroup).
constexpr int32_t kMultiMidCap = 4096;
constexpr int32_t kBfsLong = kWave * kMultiU;  // out-rows a BFS level cuts up for the wavefronts

struct MultiEntry {
    int64_t vbase;  // first vertex of the graph in the vertex arenas (x, level, parent)
    int64_t obase;  // first entry of the graph's n+1 offsets in the offset arenas
    int64_t ebase;  // first slot of the graph in the index arenas
    int32_t n;
    int32_t nnz;
};

struct MultiArgs {
    const MultiEntry* table;  // LPT order
    int32_t count;
    const int32_t* off;       // per graph: n+1 local offsets, graphs back to back
    const uint16_t* idx;      // local vertex ids (below 16384, so 16 bits hold them)
    const int32_t* in_off;
    const uint16_t* in_idx;
    int32_t pr_dir;
    int32_t pr_iters;
    float f;
    float* x;                 // PageRank output, arena of vertices
    float* c_scratch;         // push: contributions, arena of vertices
    int32_t bfs_policy;       // -1: no BFS
    int32_t root;             // local root of every graph
    float alpha, beta;
    int32_t* level;
    int32_t* parent;
    const int32_t* err;       // set by k_multi_check when the arena is malformed
    int32_t big, mid;         // row-length thresholds of the wavefront and middle groups
};

__device__ __forceinline__ uint32_t bit_of(const uint32_t* bm, int32_t v) { return (bm[v >> 5] >> (v & 31)) & 1u; }

// U slots j0, j0 + STRIDE, ... of a row ending at re (j0 < re) added to an
// FP64 sum in slot order.  The index loads are clamped to the row's last
// slot and the LDS gathers issued together, so neither waits on the one
// before; slots past the row's end read the zero word s_zero.
template <int STRIDE, int U, typename I>
__device__ __forceinline__ void gather_row_slots(const I* __restrict__ ids, const float* s_c, const float* s_zero,
                                                 slot_t j0, slot_t re, double& acc) {
    const char* base = reinterpret_cast<const char*>(ids);
    const float* src[U];
#pragma unroll
    for (int k = 0; k < U; ++k) {
        const uint32_t boff = slot_at(j0, k * STRIDE, re) * (uint32_t)sizeof(I);
        const uint32_t id = *reinterpret_cast<const I*>(base + boff);
        src[k] = slot_in(j0, k * STRIDE, re) ? s_c + id : s_zero;
    }
    float cv[U];
#pragma unroll
    for (int k = 0; k < U; ++k) cv[k] = *src[k];
#pragma unroll
    for (int k = 0; k < U; ++k) acc += (double)cv[k];
}

// Validates the arena before any sweep reads it, one workgroup per graph:
// the graph's n+1 offsets start at 0, never decrease and end at its nnz, and
// each of its nnz local ids lies below its n.  Both adjacencies are checked
// unless they alias.  Every read stays inside the graph's own offsets and
// slots, so a malformed arena is reported (PP_E_GRAPH), never walked.
// kCheckParts workgroups share a graph and keep eight loads in flight a lane
// (one 256-thread workgroup a graph, one load at a time, took 346 us over a
// scale-14 R-MAT graph).
constexpr int kCheckBlock = 256;
constexpr int kCheckParts = 8;

__device__ __forceinline__ bool offsets_ok(const int32_t* off, int32_t n, int32_t nnz, int32_t t0, int32_t step) {
    bool ok = true;
    constexpr int U = 4;
    for (int32_t v0 = t0; v0 < n; v0 += U * step) {
        int32_t a[U], b[U];
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const int32_t v = min(v0 + k * step, n - 1);
            a[k] = off[v];
            b[k] = off[v + 1];
        }
#pragma unroll
        for (int k = 0; k < U; ++k) ok &= a[k] <= b[k];
    }
    if (t0 == 0) ok &= (off[0] == 0) && (off[n] == nnz);
    return ok;
}

__device__ __forceinline__ bool ids_ok(const uint16_t* idx, int32_t n, int32_t nnz, int32_t t0, int32_t step) {
    uint32_t mx = 0;
    constexpr int U = 8;
    for (int64_t j0 = t0; j0 < nnz; j0 += (int64_t)U * step) {
#pragma unroll
        for (int k = 0; k < U; ++k) mx = max(mx, (uint32_t)idx[min(j0 + (int64_t)k * step, (int64_t)nnz - 1)]);
    }
    return nnz == 0 || mx < (uint32_t)n;
}

__global__ __launch_bounds__(kCheckBlock) void k_multi_check(const MultiEntry* __restrict__ table,
                                                             const int32_t* __restrict__ off,
                                                             const uint16_t* __restrict__ idx,
                                                             const int32_t* __restrict__ in_off,
                                                             const uint16_t* __restrict__ in_idx, int32_t* err) {
    const MultiEntry e = table[blockIdx.x];
    const int32_t t0 = blockIdx.y * kCheckBlock + threadIdx.x, step = kCheckParts * kCheckBlock;
    bool ok = offsets_ok(off + e.obase, e.n, e.nnz, t0, step) && ids_ok(idx + e.ebase, e.n, e.nnz, t0, step);
    if (in_off != off || in_idx != idx)
        ok = ok && offsets_ok(in_off + e.obase, e.n, e.nnz, t0, step) &&
             ids_ok(in_idx + e.ebase, e.n, e.nnz, t0, step);
    if (!ok) atomicOr(err, 1);
}

// Rows [r0, r1) of one graph pull: in-rows of at least `big` slots (listed in
// s_big) a wavefront each, of `mid`..`big`-1 (s_mid) ML lanes each, the others
// PG lanes each, rows spread over the wavefronts.  Every lane sums in FP64, in
// slot order; finish(u, sum, out-degree) runs in one lane of the row's owner.
// The offsets and out-degree of a group's next row load while a row is summed.
template <int PG, int ML, typename F>
__device__ __forceinline__ void multi_pull_rows(const int32_t* in_off, const uint16_t* in_idx, const int32_t* off,
                                                const float* s_c, const float* s_zero, const int32_t* s_big,
                                                int32_t nbig, const int32_t* s_mid, int32_t nmid, int32_t big,
                                                int32_t mid, int32_t r0, int32_t r1, F finish) {
    const int tid = threadIdx.x, wl = tid & (kWave - 1), wv = tid / kWave;
    constexpr int kWaves = kMultiBlock / kWave;
    // does row length d belong to the small groups?
    auto grouped = [=](int32_t d) { return !((nbig > 0 && d >= big) || (nmid > 0 && d >= mid && d < big)); };
    for (int32_t i = wv; i < nbig; i += kWaves) {
        const int32_t u = s_big[i];
        double acc = 0.0;
        const int32_t rb = in_off[u], re = in_off[u + 1];
        for (slot_t j0 = (slot_t)rb + wl; j0 < (slot_t)re; j0 += kMultiU * kWave)
            gather_row_slots<kWave, kMultiU>(in_idx, s_c, s_zero, j0, re, acc);
#pragma unroll
        for (int s = kWave / 2; s > 0; s >>= 1) acc += __shfl_xor(acc, s);
        if (wl == 0) finish(u, acc, off[u + 1] - off[u]);
    }
    {
        const int hl = wl & (ML - 1);  // lane within a middle-row group
        const int32_t mslot = (kWave / ML) * wv + wl / ML;  // its group
        constexpr int32_t mgroups = kMultiBlock / ML;
        int32_t nu = 0, nrb = 0, nre = 0, nob = 0, noe = 0;
        if (mslot < nmid) {
            nu = s_mid[mslot];
            nrb = in_off[nu];
            nre = in_off[nu + 1];
            nob = off[nu];
            noe = off[nu + 1];
        }
        for (int32_t i = mslot; i < nmid; i += mgroups) {
            const int32_t u = nu, rb = nrb, re = nre, ob = nob, oe = noe;
            if (i + mgroups < nmid) {
                nu = s_mid[i + mgroups];
                nrb = in_off[nu];
                nre = in_off[nu + 1];
                nob = off[nu];
                noe = off[nu + 1];
            }
            double acc = 0.0;
            for (slot_t j0 = (slot_t)rb + hl; j0 < (slot_t)re; j0 += kMultiU * ML)
                gather_row_slots<ML, kMultiU>(in_idx, s_c, s_zero, j0, re, acc);
#pragma unroll
            for (int s = ML / 2; s > 0; s >>= 1) acc += __shfl_xor(acc, s);
            if (hl == 0) finish(u, acc, oe - ob);
        }
    }
    const int plane = tid % PG;
    const int32_t prow0 = r0 + kWaves * ((tid % kWave) / PG) + wv;
    constexpr int32_t pgroups = kMultiBlock / PG;
    int32_t nrb = 0, nre = 0, nob = 0, noe = 0;
    if (prow0 < r1) {
        nrb = in_off[prow0];
        nre = in_off[prow0 + 1];
        nob = off[prow0];
        noe = off[prow0 + 1];
    }
    for (int32_t u = prow0; u < r1; u += pgroups) {
        double acc = 0.0;
        const int32_t rb = nrb, re = nre, ob = nob, oe = noe;
        if (u + pgroups < r1) {
            nrb = in_off[u + pgroups];
            nre = in_off[u + pgroups + 1];
            nob = off[u + pgroups];
            noe = off[u + pgroups + 1];
        }
        if (!grouped(re - rb)) continue;  // group-uniform
        for (slot_t j0 = (slot_t)rb + plane; j0 < (slot_t)re; j0 += kMultiPullU * PG)
            gather_row_slots<PG, kMultiPullU>(in_idx, s_c, s_zero, j0, re, acc);
#pragma unroll
        for (int s = PG / 2; s > 0; s >>= 1) acc += __shfl_xor(acc, s);
        if (plane == 0) finish(u, acc, oe - ob);
    }
}

// Lists the long and middle rows of [r0, r1) (roff: the sweep's direction); a
// list that would overflow counts as empty, its rows stay with the small
// groups.  Workgroup-collective.
__device__ __forceinline__ int2 multi_lists(const int32_t* roff, int32_t r0, int32_t r1, int32_t big, int32_t mid,
                                            int32_t* s_big, int32_t big_cap, int32_t* s_mid, int32_t mid_cap,
                                            int32_t* s_n) {
    if (threadIdx.x < 2) s_n[threadIdx.x] = 0;
    __syncthreads();
    for (int32_t u = r0 + (int32_t)threadIdx.x; u < r1; u += kMultiBlock) {
        const int32_t d = roff[u + 1] - roff[u];
        if (d >= big) {
            const int32_t at = atomicAdd(&s_n[0], 1);
            if (at < big_cap) s_big[at] = u;
        } else if (d >= mid) {
            const int32_t at = atomicAdd(&s_n[1], 1);
            if (at < mid_cap) s_mid[at] = u;
        }
    }
    __syncthreads();
    return make_int2(s_n[0] <= big_cap ? s_n[0] : 0, s_n[1] <= mid_cap ? s_n[1] : 0);
}

// ------------------------------------------------------- shared PageRank steps
// A workgroup's part of one graph: rows [r0, r1).  The host gives shares of the
// graph's cost (kStepGraphCost, kStepRowCost a row and one a slot);
// k_multi_pieces turns them into rows once per call.
struct MultiPiece {
    int32_t entry;   // of the graph table
    int32_t r0, r1;  // costs, then rows
};
constexpr int32_t kStepGroups = 256;  // workgroups of a step, one a compute unit (512: 45 us against 40)
// A launch costs a step about 14 us whatever is in it, and a workgroup of k_multi
// sweeps this many edges in that time; four scale-13 graphs (250,000 edges the
// largest) went from 1.57 to 0.37 ms, 64 of scales 8-12 from 0.83 to 0.38.
constexpr int32_t kStepEdges = 49152;
// What a row and the beginning of a graph cost in slots.  Beginning a graph is a
// chain of loads (its rows' offsets, the stage, the lists, the first ids) some
// 8 us long: with shares of edges alone the workgroups that got 14 small graphs
// took the whole step (74 us; 50, 40, 41 and 40 at 4096, 8192, 16384 and 32768;
// rows at 2, 8 and 16: 80, 74 and 69 without it, 43 and 40 at 8 and 16 with it).
constexpr int32_t kStepGraphCost = 8192;
constexpr int32_t kStepRowCost = 16;

// Whether shared steps pay (cost: of every graph, largest first, as k_multi_pieces
// divides it).  In the one launch a sweep ends with the workgroup of the largest
// graph, or with the compute unit that takes most graphs: at least k graphs of the
// (256 (k - 1) + 1)-th largest's cost.  A shared step is kStepLaunch of launch and
// then its 256th of everything, a quarter slower than one workgroup that keeps its
// graph in LDS.  One graph of 2^s vertices among others, 20 steps pulled, one
// launch / shared: 10,000 of 2^5, s = 12 / 13 / 14 1.70 / 1.84 / 2.94 ms against 3.0;
// 2,000 of 2^9, s = 12 / 13 0.85 / 1.51 against 1.32; 300 of 2^12 1.40 / 1.22; 600 of
// 2^13 4.26 / 4.73, pushed (where the one launch takes a quarter longer) 5.52 / 4.96.
constexpr int64_t kStepLaunch = 63000;
template <typename Cost>
static bool steps_pay(int32_t count, int64_t total, bool push, Cost cost) {
    int64_t sweep = 0;
    for (int32_t i = 0, k = 1; i < count; i += kStepGroups, ++k) sweep = std::max(sweep, k * cost(i));
    const int64_t quota = total / kStepGroups;
    return sweep + (push ? sweep / 4 : 0) > kStepLaunch + quota + quota / 4;
}

// First row before which the graph, rows and slots cost t or more.
__global__ void k_multi_pieces(const MultiEntry* __restrict__ table, const int32_t* __restrict__ in_off, int32_t count,
                               MultiPiece* __restrict__ pc, const int32_t* __restrict__ err,
                               unsigned long long* __restrict__ marks) {
    const int32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i == 0) *marks = 0ull;
    if (i >= count || *err) return;
    const MultiEntry e = table[pc[i].entry];
    const int32_t* off = in_off + e.obase;
    auto row = [&](int32_t t) {
        int32_t lo = 0, hi = e.n;
        while (lo < hi) {
            const int32_t m = (lo + hi) >> 1;
            if (kStepGraphCost + (int64_t)off[m] + (int64_t)kStepRowCost * m >= t) hi = m;
            else lo = m + 1;
        }
        return lo;
    };
    const int32_t t0 = pc[i].r0, t1 = pc[i].r1;
    pc[i].r0 = t0 <= 0 ? 0 : row(t0);
    pc[i].r1 = t1 == INT32_MAX ? e.n : row(t1);
}

// 64 bits that mark an edge, in one of a pair's two directions: the finalizer of
// MurmurHash3 (Appleby) on the ids, 28 bits, under two seeds of the graph.  Two lists
// hold the same edges when the sums of their marks agree, and other lists agree
// with probability 2^-64.
__device__ __forceinline__ uint32_t mix32(uint32_t h) {
    h ^= h >> 16;
    h *= 0x85EBCA6Bu;
    h ^= h >> 13;
    h *= 0xC2B2AE35u;
    return h ^ (h >> 16);
}
__device__ __forceinline__ uint64_t edge_mark(uint32_t s0, uint32_t s1, int32_t v, int32_t u) {
    const uint32_t key = ((uint32_t)v << 14) | (uint32_t)u;
    return ((uint64_t)mix32(key ^ s0) << 32) | mix32(key + s1);
}

// Sum of mark(row, id) over the slots of rows [r0, r1): a thread takes eight
// consecutive slots and finds the first one's row among the offsets, staged in
// s_off (sixteen lanes a row, offsets and ids loaded row by row, took ten times
// as long).  Workgroup-collective.
template <typename F>
__device__ __forceinline__ uint64_t sum_marks(const int32_t* off, const uint16_t* idx, int32_t r0, int32_t r1,
                                              int32_t* s_off, F mark) {
    constexpr int U = 8;
    __syncthreads();  // the previous rows are done with
    for (int32_t i = threadIdx.x; i <= r1 - r0; i += kMultiBlock) s_off[i] = off[r0 + i];
    __syncthreads();
    uint64_t h = 0;
    const int32_t first = s_off[0], count = s_off[r1 - r0] - first;
    for (int64_t j0 = (int64_t)threadIdx.x * U; j0 < count; j0 += (int64_t)kMultiBlock * U) {
        const int32_t live = (int32_t)min((int64_t)U, count - j0), j = first + (int32_t)j0;
        int32_t id[U];
#pragma unroll
        for (int k = 0; k < U; ++k) id[k] = idx[j + min(k, live - 1)];
        int32_t lo = 0, hi = r1 - r0;  // the last row that begins at or before slot j
        while (hi - lo > 1) {
            const int32_t m = (lo + hi) >> 1;
            if (s_off[m] <= j) lo = m;
            else hi = m;
        }
#pragma unroll
        for (int k = 0; k < U; ++k) {
            if (k >= live) break;
            while (s_off[lo + 1] <= j + k) ++lo;
            h += mark(r0 + lo, id[k]);
        }
    }
    return h;
}

// Whether the in-arrays hold the transpose of every graph: *marks ends at zero
// where they do.  Steps that sum what a push sends where it arrives need it; a
// caller who pushes directed graphs may have no in-arrays and pass the out-arrays
// twice.  128 R-MAT graphs of scales 8-14: 1,058 -> 1,114 us a pushed call.
__global__ __launch_bounds__(kMultiBlock) void k_multi_match(const MultiEntry* __restrict__ table,
                                                             const MultiPiece* __restrict__ pieces,
                                                             const int32_t* __restrict__ wg,
                                                             const int32_t* __restrict__ off,
                                                             const uint16_t* __restrict__ idx,
                                                             const int32_t* __restrict__ in_off,
                                                             const uint16_t* __restrict__ in_idx,
                                                             unsigned long long* marks, const int32_t* err) {
    extern __shared__ int32_t s_rows[];  // [largest n + 1]
    __shared__ unsigned long long s_h;
    if (*err) return;
    if (threadIdx.x == 0) s_h = 0ull;
    __syncthreads();
    uint64_t h = 0;
    const bool same = in_off == off && in_idx == idx;
    for (int32_t p = wg[blockIdx.x]; p < wg[blockIdx.x + 1]; ++p) {
        const MultiPiece pc = pieces[p];
        const MultiEntry e = table[pc.entry];
        if (pc.r0 >= pc.r1) continue;
        const uint32_t s0 = mix32(2u * (uint32_t)pc.entry + 1u), s1 = mix32(2u * (uint32_t)pc.entry + 2u);
        if (same) {  // as often v -> u as u -> v
            h += sum_marks(off + e.obase, idx + e.ebase, pc.r0, pc.r1, s_rows, [=](int32_t v, int32_t u) {
                const uint64_t m = edge_mark(s0, s1, min(v, u), max(v, u));
                return v < u ? m : v > u ? ~m + 1u : 0u;
            });
        } else {
            h += sum_marks(off + e.obase, idx + e.ebase, pc.r0, pc.r1, s_rows,
                           [=](int32_t v, int32_t u) { return edge_mark(s0, s1, v, u); });
            h -= sum_marks(in_off + e.obase, in_idx + e.ebase, pc.r0, pc.r1, s_rows,
                           [=](int32_t u, int32_t v) { return edge_mark(s0, s1, v, u); });
        }
    }
#pragma unroll
    for (int s = kWave / 2; s > 0; s >>= 1) h += __shfl_xor((unsigned long long)h, s);
    if ((threadIdx.x & (kWave - 1)) == 0) atomicAdd(&s_h, (unsigned long long)h);
    __syncthreads();
    if (threadIdx.x == 0 && s_h) atomicAdd(marks, s_h);
}

struct StepArgs {
    const MultiEntry* table;
    const MultiPiece* pc;
    const int32_t* wg;       // first piece of every workgroup [kStepGroups + 1]
    const int32_t* off;
    const int32_t* in_off;
    const uint16_t* in_idx;
    const float* c;          // contributions; NULL: those of x_0 = 1/n
    float* c_next;           // NULL after the last step
    float* x;                // last step
    const int32_t* err;
    float f;
    int32_t big, mid;        // row-length thresholds of the wavefront and middle groups
};

// One PageRank step of every graph: a workgroup stages the contributions of a
// piece's graph in LDS and pulls the piece's rows as k_multi does (the pushing
// form too, where the in-arrays are the transpose: an FP64 sum over the in-edges
// is what the FP64 adds of the out-edges come to, rounded once).  Bound by latency:
// the pieces' rows of a 128-graph batch are 32 MB of ids, 5 us at the rate of
// memory.  Laying the gathered values down in slot order and summing rows from
// there took 73 to 100 us a step against 74 of this form, before the shares knew
// what a graph costs.
template <int PG, int ML>
__global__ __launch_bounds__(kMultiBlock) void k_multi_step(StepArgs a) {
    extern __shared__ __align__(16) float s_c[];  // [largest n]
    __shared__ int32_t s_big[kMultiBigCap];
    __shared__ int32_t s_mid[kMultiMidCap];
    __shared__ int32_t s_n[2];
    __shared__ float s_zero;
    if (*a.err) return;
    const int tid = threadIdx.x;
    if (tid == 0) s_zero = 0.f;
    const int32_t p1 = a.wg[blockIdx.x + 1];
    int32_t staged = -1;
    for (int32_t p = a.wg[blockIdx.x]; p < p1; ++p) {
        const MultiPiece pc = a.pc[p];
        const MultiEntry e = a.table[pc.entry];
        const int32_t* off = a.off + e.obase;
        const int32_t* in_off = a.in_off + e.obase;
        const int32_t n = e.n;
        if (pc.r0 >= pc.r1) continue;
        __syncthreads();  // the previous piece is done with the stage and the lists
        if (pc.entry != staged) {
            constexpr int V = 8;
            for (int32_t u0 = tid; u0 < n; u0 += V * kMultiBlock) {
                float v[V];
                int32_t d[V];
#pragma unroll
                for (int k = 0; k < V; ++k) {
                    const int32_t u = min(u0 + k * kMultiBlock, n - 1);
                    if (a.c) v[k] = a.c[e.vbase + u];
                    else d[k] = off[u + 1] - off[u];
                }
#pragma unroll
                for (int k = 0; k < V; ++k)
                    if (u0 + k * kMultiBlock < n)
                        s_c[u0 + k * kMultiBlock] = a.c ? v[k] : d[k] > 0 ? a.f * (1.0f / (float)n) / (float)d[k] : 0.f;
            }
            staged = pc.entry;
        }
        const float base = (1.0f - a.f) / (float)n;
        const int2 cnt = multi_lists(in_off, pc.r0, pc.r1, a.big, a.mid, s_big, kMultiBigCap, s_mid, kMultiMidCap, s_n);
        multi_pull_rows<PG, ML>(in_off, a.in_idx + e.ebase, off, s_c, &s_zero, s_big, cnt.x, s_mid, cnt.y, a.big, a.mid,
                                pc.r0, pc.r1, [&](int32_t u, double acc, int32_t d) {
                                    const float y = (float)((double)base + acc);
                                    if (a.c_next) a.c_next[e.vbase + u] = d > 0 ? a.f * y / (float)d : 0.f;
                                    else a.x[e.vbase + u] = y;
                                });
    }
}

template <int PG, int ML>
__global__ __launch_bounds__(kMultiBlock) void k_multi(MultiArgs a) {
    extern __shared__ float lds[];
    __shared__ int32_t s_cnt[4];
    __shared__ int64_t s_m[2];
    const int32_t gi = blockIdx.x;
    if (gi >= a.count || *a.err) return;  // a malformed arena is never walked
    const int32_t big = a.big, mid = a.mid;
    const MultiEntry e = a.table[gi];
    const int32_t n = e.n;
    const int32_t* off = a.off + e.obase;
    const uint16_t* idx = a.idx + e.ebase;
    const int32_t* in_off = a.in_off + e.obase;
    const uint16_t* in_idx = a.in_idx + e.ebase;
    const int tid = threadIdx.x;
    const int lane = tid % kMultiGroup;
    const int grp = tid / kMultiGroup;
    constexpr int groups = kMultiBlock / kMultiGroup;
    constexpr int kWaves = kMultiBlock / kWave;
    const int wl = tid & (kWave - 1), wv = tid / kWave;
    // PageRank rows of the small groups: consecutive rows go to different
    // wavefronts (rows 16 q + w + k * groups for group q of wavefront w), so
    // neighbouring ids -- the hubs of an R-MAT graph -- are spread out
    const int32_t row0 = kWaves * ((tid % kWave) / kMultiGroup) + wv;

    // ---------------------------------------------------------------- PageRank
    __shared__ int32_t s_big[kMultiBigCap];
    __shared__ int32_t s_mid[kMultiMidCap];
    __shared__ int32_t s_n[2];
    __shared__ float s_zero;
    if (a.pr_iters > 0) {
        const float base = (1.0f - a.f) / (float)n;
        // the long rows of the sweep's direction (in-rows pull, out-rows push)
        const int32_t* roff = (a.pr_dir == PP_PULL) ? in_off : off;
        if (tid == 0) s_zero = 0.f;
        const int2 cnt = multi_lists(roff, 0, n, big, mid, s_big, kMultiBigCap, s_mid, kMultiMidCap, s_n);
        const int32_t nbig = cnt.x, nmid = cnt.y;
        // does row length d belong to the small groups?
        auto grouped = [=](int32_t d) {
            return !((nbig > 0 && d >= big) || (nmid > 0 && d >= mid && d < big));
        };
        const int hl = wl & (ML - 1);  // lane within a middle-row group
        const int32_t mslot = (kWave / ML) * wv + wl / ML;  // its group
        constexpr int32_t mgroups = kMultiBlock / ML;
        if (a.pr_dir == PP_PULL) {
            float* s_c = lds;       // contributions of the current iterate
            float* s_y = lds + n;   // contributions of the next one
            for (int32_t u = tid; u < n; u += kMultiBlock) {
                const int32_t d = off[u + 1] - off[u];
                s_c[u] = d > 0 ? a.f * (1.0f / (float)n) / (float)d : 0.f;
            }
            __syncthreads();
            for (int32_t t = 0; t < a.pr_iters; ++t) {
                const bool last = (t == a.pr_iters - 1);
                multi_pull_rows<PG, ML>(in_off, in_idx, off, s_c, &s_zero, s_big, nbig, s_mid, nmid, big, mid, 0, n,
                                        [&](int32_t u, double acc, int32_t d) {
                                            const float y = (float)((double)base + acc);
                                            s_y[u] = d > 0 ? a.f * y / (float)d : 0.f;
                                            if (last) a.x[e.vbase + u] = y;
                                        });
                __syncthreads();
                float* tmp = s_c;
                s_c = s_y;
                s_y = tmp;
            }
        } else {
            // every out-edge adds the source's contribution to an FP64 LDS
            // accumulator (the order of the adds is arbitrary); contributions
            // live in the global scratch arena
            double* s_acc = reinterpret_cast<double*>(lds);
            float* c = a.c_scratch + e.vbase;
            for (int32_t u = tid; u < n; u += kMultiBlock) {
                const int32_t d = off[u + 1] - off[u];
                c[u] = d > 0 ? a.f * (1.0f / (float)n) / (float)d : 0.f;
                s_acc[u] = 0.0;
            }
            __syncthreads();
            for (int32_t t = 0; t < a.pr_iters; ++t) {
                const bool last = (t == a.pr_iters - 1);
                // long out-rows: a whole wavefront each
                for (int32_t i = wv; i < nbig; i += kWaves) {
                    const int32_t v = s_big[i];
                    const float cv = c[v];
                    if (cv == 0.f) continue;
                    const int32_t rb = off[v], re = off[v + 1];
                    for (slot_t j0 = (slot_t)rb + wl; j0 < (slot_t)re; j0 += kMultiU * kWave) {
                        int32_t ii[kMultiU];
#pragma unroll
                        for (int k = 0; k < kMultiU; ++k) {
                            ii[k] = slot_in(j0, k * kWave, re) ? idx[j0 + k * kWave] : -1;
                        }
#pragma unroll
                        for (int k = 0; k < kMultiU; ++k)
                            if (ii[k] >= 0) atomicAdd(&s_acc[ii[k]], (double)cv);
                    }
                }
                // middle out-rows: 16 lanes each
                {
                    int32_t nv = 0, nb = 0, ne = 0;
                    float ncv = 0.f;
                    if (mslot < nmid) {
                        nv = s_mid[mslot];
                        ncv = c[nv];
                        nb = off[nv];
                        ne = off[nv + 1];
                    }
                    for (int32_t i = mslot; i < nmid; i += mgroups) {
                        const float cv = ncv;
                        const int32_t rb = nb, re = ne;
                        if (i + mgroups < nmid) {
                            nv = s_mid[i + mgroups];
                            ncv = c[nv];
                            nb = off[nv];
                            ne = off[nv + 1];
                        }
                        if (cv == 0.f) continue;
                        for (slot_t j0 = (slot_t)rb + hl; j0 < (slot_t)re; j0 += kMultiU * ML) {
                            int32_t ii[kMultiU];  // clamped to the row's last slot
#pragma unroll
                            for (int k = 0; k < kMultiU; ++k)
                                ii[k] = idx[slot_at(j0, k * ML, re)];
#pragma unroll
                            for (int k = 0; k < kMultiU; ++k)
                                if (slot_in(j0, k * ML, re)) atomicAdd(&s_acc[ii[k]], (double)cv);
                        }
                    }
                }
                // two rows per group and round (v and v + groups), their index
                // loads issued together; the contributions and offsets of the
                // group's next two rows load while these are scattered
                float pc[2];
                int32_t pb[2], pe[2];
#pragma unroll
                for (int r = 0; r < 2; ++r) {
                    const int32_t w = row0 + r * groups;
                    pc[r] = 0.f;
                    pb[r] = pe[r] = 0;
                    if (w < n) {
                        pc[r] = c[w];
                        pb[r] = off[w];
                        pe[r] = off[w + 1];
                    }
                }
                for (int32_t v = row0; v < n; v += 2 * groups) {
                    float cv[2];
                    int32_t rb[2], re[2];
#pragma unroll
                    for (int r = 0; r < 2; ++r) {
                        cv[r] = pc[r];
                        rb[r] = pb[r];
                        re[r] = pe[r];
                        const int32_t w = v + (2 + r) * groups;
                        if (w < n) {
                            pc[r] = c[w];
                            pb[r] = off[w];
                            pe[r] = off[w + 1];
                        }
                        // nothing to scatter here: past the graph, a zero
                        // contribution, or a long row (done above)
                        if (v + r * groups >= n || cv[r] == 0.f || !grouped(re[r] - rb[r])) re[r] = rb[r];
                    }
                    const slot_t len = max(re[0] - rb[0], re[1] - rb[1]);
                    for (slot_t d = lane; d < len; d += kMultiU * kMultiGroup) {
                        // clamped into [0, re - 1]: a finished or empty row
                        // rereads a valid slot (the graph has edges, or len = 0)
                        int32_t ii[2][kMultiU];
#pragma unroll
                        for (int r = 0; r < 2; ++r)
#pragma unroll
                            for (int k = 0; k < kMultiU; ++k)
                                ii[r][k] = idx[re[r] > 0 ? slot_at((slot_t)rb[r] + d, k * kMultiGroup, re[r]) : 0u];
#pragma unroll
                        for (int r = 0; r < 2; ++r)
#pragma unroll
                            for (int k = 0; k < kMultiU; ++k)
                                if (slot_in((slot_t)rb[r] + d, k * kMultiGroup, re[r])) atomicAdd(&s_acc[ii[r][k]], (double)cv[r]);
                    }
                }
                __syncthreads();
                for (int32_t u = tid; u < n; u += kMultiBlock) {
                    const float y = base + (float)s_acc[u];
                    const int32_t d = off[u + 1] - off[u];
                    c[u] = d > 0 ? a.f * y / (float)d : 0.f;
                    s_acc[u] = 0.0;
                    if (last) a.x[e.vbase + u] = y;
                }
                __syncthreads();
            }
        }
    }

    // ---------------------------------------------------------------- BFS
    if (a.bfs_policy < 0) return;
    const int32_t words = (n + 31) / 32;
    uint32_t* s_front = reinterpret_cast<uint32_t*>(lds);
    uint32_t* s_next = s_front + words;
    uint32_t* s_vis = s_next + words;
    const int32_t root = a.root;
    for (int32_t v = tid; v < n; v += kMultiBlock) {
        a.level[e.vbase + v] = (v == root) ? 0 : -1;
        a.parent[e.vbase + v] = (v == root) ? root : -1;
    }
    for (int32_t w = tid; w < words; w += kMultiBlock) {
        const uint32_t m = (w == (root >> 5)) ? (1u << (root & 31)) : 0u;
        s_front[w] = m;
        s_vis[w] = m;
        s_next[w] = 0u;
    }
    if (tid == 0) {
        s_cnt[0] = 1;                          // |F|
        s_m[0] = off[root + 1] - off[root];    // out-edges of F
        s_m[1] = (int64_t)(off[n] - off[root + 1] + off[root]);  // out-edges of unvisited vertices
        s_cnt[2] = PP_PUSH;                    // previous direction
        s_cnt[3] = 0;                          // previous |F|
    }
    __syncthreads();
    for (int32_t lvl = 0;; ++lvl) {
        const int32_t nf = s_cnt[0];
        if (nf == 0) break;
        const int64_t mf = s_m[0], mu = s_m[1];
        int32_t dir = a.bfs_policy;
        if (dir == PP_SWITCH) {
            if (lvl == 0 || s_cnt[2] == PP_PUSH) dir = ((double)mf > (double)mu / a.alpha) ? PP_PULL : PP_PUSH;
            else dir = ((double)nf < (double)n / a.beta && nf < s_cnt[3]) ? PP_PUSH : PP_PULL;
        }
        __syncthreads();
        if (tid == 0) {
            s_cnt[1] = 0;
            s_cnt[2] = dir;
            s_cnt[3] = nf;
        }
        if (tid < 2) s_m[tid] = 0;  // s_m[0] accumulates new out-edges; s_m[1] is recomputed below
        __syncthreads();
        int32_t my_new = 0;
        int64_t my_deg = 0;
        if (dir == PP_PUSH) {
            // frontier vertices claim unvisited out-neighbours (LDS atomic OR):
            // slots j0, j0 + stride, ... of v's row, which ends at re
            auto scatter = [&](int32_t v, slot_t j0, int32_t stride, slot_t re) {
                // index loads clamped to the row's last slot, then every
                // visited probe issued before the first claim (a probe only
                // filters: the atomic OR decides)
                int32_t ii[kMultiU];
#pragma unroll
                for (int k = 0; k < kMultiU; ++k) ii[k] = idx[slot_at(j0, k * stride, re)];
                uint32_t seen[kMultiU];
#pragma unroll
                for (int k = 0; k < kMultiU; ++k) seen[k] = s_vis[min(ii[k], n - 1) >> 5];
#pragma unroll
                for (int k = 0; k < kMultiU; ++k) {
                    const int32_t u = ii[k];
                    if (!slot_in(j0, k * stride, re) || u >= n) continue;  // ids past the graph are ignored
                    const uint32_t b = 1u << (u & 31);
                    if (seen[k] & b) continue;
                    const uint32_t old = atomicOr(&s_vis[u >> 5], b);
                    if (!(old & b)) {
                        atomicOr(&s_next[u >> 5], b);
                        a.level[e.vbase + u] = lvl + 1;
                        a.parent[e.vbase + u] = v;
                        my_new += 1;
                        my_deg += off[u + 1] - off[u];
                    }
                }
            };
            // rows of kBfsLong or more are cut into pieces of as many edges for
            // the wavefronts (four lanes on the root's row of thousands held
            // up the whole level); a full list leaves the rest to the groups
            if (tid == 0) s_n[0] = 0;
            __syncthreads();
            for (int32_t v = grp; v < n; v += groups) {
                if (!bit_of(s_front, v)) continue;
                const int32_t rb = off[v], re = off[v + 1];
                if (re - rb >= kBfsLong) {
                    int32_t at = 0;
                    if (lane == 0) at = atomicAdd(&s_n[0], 1);
                    at = __shfl(at, (tid & (kWave - 1)) - lane);
                    if (at < kMultiMidCap) {
                        if (lane == 0) s_mid[at] = v;
                        continue;
                    }
                }
                for (slot_t j0 = (slot_t)rb + lane; j0 < (slot_t)re; j0 += kMultiU * kMultiGroup) scatter(v, j0, kMultiGroup, re);
            }
            __syncthreads();
            const int32_t nlong = min(s_n[0], kMultiMidCap);
            int32_t turn = wv;  // pieces until this wavefront's next one
            for (int32_t i = 0; i < nlong; ++i) {
                const int32_t v = s_mid[i];
                const int32_t rb = off[v], re = off[v + 1];
                const int32_t np = (int32_t)(((slot_t)(re - rb) + kBfsLong - 1) / kBfsLong);
                for (; turn < np; turn += kWaves) {
                    const slot_t b = (slot_t)rb + turn * kBfsLong, pe = min((slot_t)re, b + kBfsLong);
                    if (b + wl < pe) scatter(v, b + wl, kWave, pe);
                }
                turn -= np;
            }
        } else {
            // unvisited vertices look for a frontier in-neighbour, first in stored order
            for (int32_t v = grp; v < n; v += groups) {
                if (bit_of(s_vis, v)) continue;
                const int32_t b0 = in_off[v], e0 = in_off[v + 1];
                int32_t hit = INT32_MAX;
                // kMultiU steps of kMultiGroup in-neighbours per round; the
                // first frontier member in stored order wins
                for (slot_t jb = b0; jb < (slot_t)e0 && hit == INT32_MAX; jb += kMultiU * kMultiGroup) {
                    // index loads clamped to the row's last slot, frontier words
                    // read together (ids past the graph read a valid word and
                    // are then ignored)
                    int32_t ii[kMultiU];
#pragma unroll
                    for (int k = 0; k < kMultiU; ++k)
                        ii[k] = in_idx[slot_at(jb, k * kMultiGroup + lane, e0)];
                    uint32_t fw[kMultiU];
#pragma unroll
                    for (int k = 0; k < kMultiU; ++k) fw[k] = s_front[min(ii[k], n - 1) >> 5];
                    int32_t pos = INT32_MAX;
#pragma unroll
                    for (int k = kMultiU - 1; k >= 0; --k) {
                        if (slot_in(jb, k * kMultiGroup + lane, e0) && ii[k] < n && ((fw[k] >> (ii[k] & 31)) & 1u))
                            pos = (int32_t)(jb + k * kMultiGroup + lane);
                    }
#pragma unroll
                    for (int s = kMultiGroup / 2; s > 0; s >>= 1) pos = min(pos, __shfl_xor(pos, s));
                    hit = pos;
                }
                if (hit != INT32_MAX && lane == 0) {
                    atomicOr(&s_next[v >> 5], 1u << (v & 31));  // words are shared by groups
                    a.level[e.vbase + v] = lvl + 1;
                    a.parent[e.vbase + v] = in_idx[hit];
                    my_new += 1;
                    my_deg += off[v + 1] - off[v];
                }
            }
        }
        if (my_new) {
            atomicAdd(&s_cnt[1], my_new);
            atomicAdd(reinterpret_cast<unsigned long long*>(&s_m[0]), (unsigned long long)my_deg);
        }
        __syncthreads();
        // next frontier; bottom-up discoveries become visited now
        for (int32_t w = tid; w < words; w += kMultiBlock) {
            const uint32_t nw = s_next[w];
            s_front[w] = nw;
            s_vis[w] |= nw;
            s_next[w] = 0u;
        }
        if (tid == 0) {
            s_cnt[0] = s_cnt[1];
            s_m[1] = mu - s_m[0];
        }
        __syncthreads();
    }
}

// ------------------------------------------------------------------ host side
template <int PG, int ML>
static void launch_multi_k(const MultiArgs& a, int32_t grid, size_t lds, hipStream_t st) {
    allow_dynamic_lds(reinterpret_cast<const void*>(&k_multi<PG, ML>), lds);
    hipLaunchKernelGGL((k_multi<PG, ML>), dim3(grid), dim3(kMultiBlock), lds, st, a);
}

// Calls fn with the tuned group widths as types (false: no such kernel).
template <typename F>
static bool with_widths(int32_t pg, int32_t ml, F fn) {
    auto by_ml = [&](auto pg_tag) {
        switch (ml) {
            case 8: fn(pg_tag, std::integral_constant<int, 8>{}); return true;
            case 16: fn(pg_tag, std::integral_constant<int, 16>{}); return true;
            case 32: fn(pg_tag, std::integral_constant<int, 32>{}); return true;
            default: return false;
        }
    };
    switch (pg) {
        case 1: return by_ml(std::integral_constant<int, 1>{});
        case 2: return by_ml(std::integral_constant<int, 2>{});
        case 4: return by_ml(std::integral_constant<int, 4>{});
        default: return false;
    }
}

static bool launch_multi(int32_t pg, int32_t ml, const MultiArgs& a, int32_t grid, size_t lds, hipStream_t st) {
    return with_widths(pg, ml, [&](auto p, auto m) {
        launch_multi_k<decltype(p)::value, decltype(m)::value>(a, grid, lds, st);
    });
}

// Workspace: the graph table (LPT order) and the validation error word, both
// written by one host copy, then the push contributions (one float per vertex).
// After those, where it fits, what the shared steps need: the pieces, every
// workgroup's first one and the marks' sum.
struct MultiLayout {
    size_t table, err, cbuf, base, pieces, wg, marks, total;
};

static MultiLayout multi_layout(int32_t count, int64_t total_n) {
    MultiLayout L{};
    L.table = 0;
    L.err = (size_t)std::max(count, 1) * sizeof(MultiEntry);
    L.cbuf = align_up(L.err + sizeof(int32_t), 256);
    L.base = L.cbuf + align_up((size_t)std::max<int64_t>(total_n, 1) * 4, 256);
    L.pieces = L.base;
    L.wg = L.pieces + align_up(((size_t)std::max(count, 1) + kStepGroups) * sizeof(MultiPiece), 256);
    L.marks = align_up(L.wg + (kStepGroups + 1) * sizeof(int32_t), 8);
    L.total = align_up(L.marks + sizeof(unsigned long long), 256);
    return L;
}

// Scratch of pp_multi_run_static (for callers that cannot allocate device
// memory): the graph table, the validation word and the push contributions of
// one call live in this file-scope array, of which every device the library
// runs on holds one copy for the life of the process.  Host code never passes
// the array's name to a kernel (on the host it is only a stand-in symbol): the
// device address comes from hipGetSymbolAddress, once per device.
constexpr size_t kMultiStaticBytes = PP_MULTI_STATIC_BYTES;
static __device__ __align__(256) unsigned char scratch[kMultiStaticBytes];

constexpr int kMaxDevices = 64;

// Device address of this device's copy of `scratch` (looked up on the first
// call on each device, with that device current).
static pp_status static_scratch(void** out) {
    static std::mutex mu;
    static void* ptr[kMaxDevices] = {};
    int dev = 0;
    PP_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices) return set_error(PP_E_UNSUPPORTED, "device ordinal beyond the static table");
    std::lock_guard<std::mutex> lock(mu);
    if (!ptr[dev]) {
        void* p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return hip_error(e, "hipGetSymbolAddress(scratch)");
        if (!p) return set_error(PP_E_HIP, "hipGetSymbolAddress(scratch) returned NULL");
        ptr[dev] = p;
    }
    *out = ptr[dev];
    return PP_OK;
}

}  // namespace pp

using namespace pp;

PP_EXPORT size_t pp_multi_workspace_bytes(int32_t num_graphs, int64_t total_vertices) {
    if (num_graphs < 0 || total_vertices < 0) return 0;
    return multi_layout(num_graphs, total_vertices).total;
}

namespace pp {

// The call behind pp_multi_run and pp_multi_run_static: ws is the workspace
// (caller memory, or the static scratch of this file).
static pp_status multi_run(int32_t num_graphs, const int32_t* graph_n, const int64_t* graph_nnz, const int32_t* off,
                           const uint16_t* idx, const int32_t* in_off, const uint16_t* in_idx, pp_dir pr_dir,
                           int32_t pr_iters, float f, float* x, int32_t bfs_policy, int32_t bfs_root, float alpha,
                           float beta, int32_t* level, int32_t* parent, void* ws, size_t ws_bytes, bool static_ws,
                           void* stream) {
    clear_error();
    if (num_graphs < 0) return set_error(PP_E_SIZE, "num_graphs must be >= 0");
    if (num_graphs == 0) return PP_OK;
    if (!graph_n || !graph_nnz) return set_error(PP_E_NULL, "graph_n and graph_nnz (host arrays) are required");
    if (!off || !in_off || (!ws && !static_ws)) return set_error(PP_E_NULL, "off, in_off and ws are required");
    if (pr_dir != PP_PUSH && pr_dir != PP_PULL) return set_error(PP_E_RANGE, "pr_dir must be PP_PUSH or PP_PULL");
    if (pr_iters < 0) return set_error(PP_E_RANGE, "pr_iters must be >= 0");
    if (pr_iters > 0 && !x) return set_error(PP_E_NULL, "x is required when pr_iters > 0");
    if (!(f >= 0.f && f < 1.f)) return set_error(PP_E_RANGE, "f must lie in [0, 1)");
    if (bfs_policy != -1 && bfs_policy != PP_PUSH && bfs_policy != PP_PULL && bfs_policy != PP_SWITCH)
        return set_error(PP_E_RANGE, "bfs_policy must be -1, PP_PUSH, PP_PULL or PP_SWITCH");
    if (bfs_policy >= 0 && (!level || !parent)) return set_error(PP_E_NULL, "level and parent are required for BFS");
    if (!(alpha > 0.f)) alpha = 14.f;
    if (!(beta > 0.f)) beta = 24.f;
    std::vector<MultiEntry> ent(num_graphs);
    int64_t vb = 0, eb = 0, max_n = 1, total_nnz = 0;
    for (int32_t i = 0; i < num_graphs; ++i) {
        if (graph_n[i] < 1 || graph_n[i] > kMultiMaxN)
            return set_error(PP_E_SIZE, "every graph needs 1 <= n <= 16384 vertices");
        if (graph_nnz[i] < 0 || graph_nnz[i] > INT32_MAX) return set_error(PP_E_SIZE, "graph nnz out of range");
        if (bfs_policy >= 0 && (bfs_root < 0 || bfs_root >= graph_n[i]))
            return set_error(PP_E_RANGE, "bfs_root must be a vertex of every graph");
        ent[i] = MultiEntry{vb, vb + i, eb, graph_n[i], (int32_t)graph_nnz[i]};
        vb += graph_n[i];
        eb += graph_nnz[i];
        total_nnz += graph_nnz[i];
        max_n = std::max<int64_t>(max_n, graph_n[i]);
    }
    if (total_nnz > 0 && (!idx || !in_idx)) return set_error(PP_E_NULL, "idx and in_idx are required");
    const MultiLayout ML = multi_layout(num_graphs, vb);
    if (static_ws && ML.base > kMultiStaticBytes)
        return set_error(PP_E_WORKSPACE, "pp_multi_run_static: the graphs need " + std::to_string(ML.base) +
                                             " bytes of scratch, more than its " + std::to_string(kMultiStaticBytes) +
                                             " (use pp_multi_run with a caller workspace)");
    if (static_ws) {
        pp_status st_ptr = static_scratch(&ws);
        if (st_ptr != PP_OK) return st_ptr;
        ws_bytes = kMultiStaticBytes;
    }
    if (ws_bytes < ML.base) return set_error(PP_E_WORKSPACE, "workspace too small");
    // largest graphs first (workgroups are dispatched roughly in index order)
    std::vector<int32_t> order(num_graphs);
    std::iota(order.begin(), order.end(), 0);
    std::stable_sort(order.begin(), order.end(), [&](int32_t p, int32_t q) {
        return (int64_t)ent[p].nnz + ent[p].n > (int64_t)ent[q].nnz + ent[q].n;
    });
    // the table in LPT order followed by a zero error word, copied together
    std::vector<char> head(ML.err + sizeof(int32_t), 0);
    MultiEntry* dev = reinterpret_cast<MultiEntry*>(head.data());
    for (int32_t i = 0; i < num_graphs; ++i) dev[i] = ent[order[i]];
    int dev_id = 0, lds_cu = 0;
    PP_HIP(hipGetDevice(&dev_id));
    PP_HIP(hipDeviceGetAttribute(&lds_cu, hipDeviceAttributeMaxSharedMemoryPerBlock, dev_id));
    const size_t lds = std::max<size_t>((size_t)max_n * 8, (size_t)3 * ((max_n + 31) / 32) * 4);
    if (lds > (size_t)lds_cu) return set_error(PP_E_UNSUPPORTED, "graphs too large for one workgroup's LDS");
    hipStream_t st = static_cast<hipStream_t>(stream);
    MultiEntry* table = static_cast<MultiEntry*>(ws);
    int32_t* err = reinterpret_cast<int32_t*>(static_cast<char*>(ws) + ML.err);
    PP_HIP(hipMemcpyAsync(table, head.data(), head.size(), hipMemcpyHostToDevice, st));
    const uint16_t* idx_chk = idx ? idx : in_idx;  // both NULL only when no graph has edges
    const uint16_t* in_idx_chk = in_idx ? in_idx : idx;
    hipLaunchKernelGGL(k_multi_check, dim3(num_graphs, kCheckParts), dim3(kCheckBlock), 0, st, (const MultiEntry*)table, off,
                       idx_chk, in_off, in_idx_chk, err);
    PP_LAUNCH_CHECK("k_multi_check");
    MultiArgs a;
    a.table = table;
    a.count = num_graphs;
    a.off = off;
    a.idx = idx;
    a.in_off = in_off;
    a.in_idx = in_idx;
    a.pr_dir = pr_dir;
    a.pr_iters = pr_iters;
    a.f = f;
    a.x = x;
    a.c_scratch = reinterpret_cast<float*>(static_cast<char*>(ws) + ML.cbuf);
    a.bfs_policy = bfs_policy;
    a.root = bfs_root;
    a.alpha = alpha;
    a.beta = beta;
    a.level = level;
    a.parent = parent;
    a.err = err;
    const Tuning& t = tuning();
    a.big = t.multi_big;
    a.mid = t.multi_mid;
    // where a few graphs are large: the steps shared among all workgroups first,
    // then (with no steps left to it) the launch below for the searches.
    // (The costs of a graph of 2^30 edges or more do not fit a piece.)
    std::vector<MultiPiece> pieces;
    std::vector<int32_t> wg;
    auto cost_of = [&](int32_t i) { return kStepGraphCost + dev[i].nnz + kStepRowCost * (int64_t)dev[i].n; };
    const int64_t total = kStepGraphCost * (int64_t)num_graphs + total_nnz + kStepRowCost * vb;
    if (pr_iters > 0 && dev[0].nnz > kStepEdges && dev[0].nnz < (1 << 30) && ws_bytes >= ML.total &&
        steps_pay(num_graphs, total, pr_dir == PP_PUSH, cost_of)) {
        int64_t run = 0;
        const int64_t quota = std::max<int64_t>(1, (total + kStepGroups - 1) / kStepGroups);
        wg.push_back(0);
        for (int32_t i = 0; i < num_graphs; ++i) {
            const int64_t cost = cost_of(i);
            int64_t at = 0;
            while (at < cost) {
                const int64_t take = std::min(cost - at, quota * (int64_t)wg.size() - run);
                const int64_t end = at + take;
                pieces.push_back(MultiPiece{i, (int32_t)at, end >= cost ? INT32_MAX : (int32_t)end});
                at = end;
                run += take;
                if (run >= quota * (int64_t)wg.size() && (int32_t)wg.size() < kStepGroups)
                    wg.push_back((int32_t)pieces.size());
            }
        }
        while ((int32_t)wg.size() <= kStepGroups) wg.push_back((int32_t)pieces.size());
    }
    MultiPiece* const pc = reinterpret_cast<MultiPiece*>(static_cast<char*>(ws) + ML.pieces);
    int32_t* const wg_dev = reinterpret_cast<int32_t*>(static_cast<char*>(ws) + ML.wg);
    bool shared = !pieces.empty();
    if (shared) {
        unsigned long long* marks = reinterpret_cast<unsigned long long*>(static_cast<char*>(ws) + ML.marks);
        PP_HIP(hipMemcpyAsync(pc, pieces.data(), pieces.size() * sizeof(MultiPiece), hipMemcpyHostToDevice, st));
        PP_HIP(hipMemcpyAsync(wg_dev, wg.data(), wg.size() * sizeof(int32_t), hipMemcpyHostToDevice, st));
        hipLaunchKernelGGL(k_multi_pieces, dim3(ceil_div((int64_t)pieces.size(), 64)), dim3(64), 0, st,
                           (const MultiEntry*)table, in_off, (int32_t)pieces.size(), pc, (const int32_t*)err, marks);
        PP_LAUNCH_CHECK("k_multi_pieces");
        if (pr_dir == PP_PUSH) {
            const size_t rows_lds = ((size_t)max_n + 1) * sizeof(int32_t);
            allow_dynamic_lds(reinterpret_cast<const void*>(&k_multi_match), rows_lds);
            hipLaunchKernelGGL(k_multi_match, dim3(kStepGroups), dim3(kMultiBlock), rows_lds, st, (const MultiEntry*)table,
                               (const MultiPiece*)pc, (const int32_t*)wg_dev, off, idx, in_off, in_idx, marks,
                               (const int32_t*)err);
            PP_LAUNCH_CHECK("k_multi_match");
            unsigned long long left = 0;
            PP_HIP(hipMemcpyAsync(&left, marks, sizeof(left), hipMemcpyDeviceToHost, st));
            PP_HIP(hipStreamSynchronize(st));
            shared = left == 0;
        }
    }
    if (shared) {
        StepArgs sa{};
        sa.table = table;
        sa.pc = pc;
        sa.wg = wg_dev;
        sa.off = off;
        sa.in_off = in_off;
        sa.in_idx = in_idx;
        sa.err = err;
        sa.f = f;
        sa.big = a.big;
        sa.mid = a.mid;
        const size_t step_lds = (size_t)max_n * sizeof(float);
        bool known = true;
        // the contributions go back and forth between the scratch and x, so
        // that the last step, which writes x, reads the scratch
        float* buf[2] = {a.c_scratch, x};
        for (int32_t i = 0; i < pr_iters; ++i) {
            const int32_t to_end = pr_iters - 1 - i;
            sa.c = i == 0 ? nullptr : buf[to_end & 1];
            sa.c_next = to_end == 0 ? nullptr : buf[(to_end - 1) & 1];
            sa.x = x;
            known = with_widths(t.multi_pull_group, t.multi_mid_lanes, [&](auto p, auto m) {
                auto kern = &k_multi_step<decltype(p)::value, decltype(m)::value>;
                if (i == 0) allow_dynamic_lds(reinterpret_cast<const void*>(kern), step_lds);
                hipLaunchKernelGGL(kern, dim3(kStepGroups), dim3(kMultiBlock), step_lds, st, sa);
            });
        }
        if (!known) return set_error(PP_E_RANGE, "many-graph tuning: unsupported group widths");
        PP_LAUNCH_CHECK("k_multi_step");
        a.pr_iters = 0;
    }
    const size_t lds_run = a.pr_iters > 0 ? lds : (size_t)3 * ((max_n + 31) / 32) * 4;
    if ((a.pr_iters > 0 || bfs_policy >= 0) && !launch_multi(t.multi_pull_group, t.multi_mid_lanes, a, num_graphs, lds_run, st))
        return set_error(PP_E_RANGE, "many-graph tuning: unsupported group widths");
    PP_LAUNCH_CHECK("k_multi");
    int32_t herr = 0;
    PP_HIP(hipMemcpyAsync(&herr, err, sizeof(herr), hipMemcpyDeviceToHost, st));
    // the host table must outlive the asynchronous copy
    PP_HIP(hipStreamSynchronize(st));
    if (herr) return set_error(PP_E_GRAPH, "a graph of the arena has malformed offsets or an id past its n");
    return PP_OK;
}

}  // namespace pp

PP_EXPORT pp_status pp_multi_run(int32_t num_graphs, const int32_t* graph_n, const int64_t* graph_nnz,
                                 const int32_t* off, const uint16_t* idx, const int32_t* in_off,
                                 const uint16_t* in_idx, pp_dir pr_dir, int32_t pr_iters, float f, float* x,
                                 int32_t bfs_policy, int32_t bfs_root, float alpha, float beta, int32_t* level,
                                 int32_t* parent, void* ws, size_t ws_bytes, void* stream) {
    return multi_run(num_graphs, graph_n, graph_nnz, off, idx, in_off, in_idx, pr_dir, pr_iters, f, x, bfs_policy,
                     bfs_root, alpha, beta, level, parent, ws, ws_bytes, false, stream);
}

PP_EXPORT pp_status pp_multi_run_static(int32_t num_graphs, const int32_t* graph_n, const int64_t* graph_nnz,
                                        const int32_t* off, const uint16_t* idx, const int32_t* in_off,
                                        const uint16_t* in_idx, pp_dir pr_dir, int32_t pr_iters, float f, float* x,
                                        int32_t bfs_policy, int32_t bfs_root, float alpha, float beta,
                                        int32_t* level, int32_t* parent, void* stream) {
    return multi_run(num_graphs, graph_n, graph_nnz, off, idx, in_off, in_idx, pr_dir, pr_iters, f, x, bfs_policy,
                     bfs_root, alpha, beta, level, parent, nullptr, 0, true, stream);
}
