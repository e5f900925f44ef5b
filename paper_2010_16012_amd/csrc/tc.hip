// Triangle counting in its pushing and pulling forms (Sec. 3.2; Sec. 4.2
// listing).  For every vertex v and every pair of neighbours (w1, w2) with w2
// adjacent to w1, the pulling form credits v and the pushing form credits w1
// (an integer fetch-and-add on another vertex's counter); halving gives the
// triangles per vertex.  Here the pairs of one (v, w1) edge are counted
// together: |N(v) ∩ N(w1)| over sorted rows.
//
// |N(v) ∩ N(w)| does not depend on the order of v and w, so k_tc_count forms it
// once per pair, at the endpoint with the longer row (the owner, ties by id):
// the owner's row is a bitmap or a list in LDS and the shorter row is streamed
// against it, sum over the edges of min(d(v), d(w)) tests in all.  The stream of N(w)
// meets the owner itself where the reverse edge is stored, so the count is
// written to both slots without a search.  k_tc_slices then sums the counts of
// each row's slots; a slot without one (two short rows, a directed edge to a longer
// row that has no edge back) is intersected there.  What bounds it: LDS bit tests and
// the barriers between a slice's rows.  R-MAT 16 (163M tests): 0.34 ms a call,
// against 20.3 ms with a wavefront per 256 edges that searched or merged both
// directions of every pair in global memory.
//
// Work decomposition: the edge array is cut into slices of kTcSlice edges,
// one workgroup (counting) or wavefront (summing) each, so the load is
// balanced whatever the degrees.
//
// Pull writes each vertex's counter exactly once: counts are reduced over the
// lanes of a row inside the slice (segmented scan); a row that crosses slice
// boundaries leaves partial sums (the last segment of its first slice, the
// first segment of each later slice) that k_tc_fix adds in a fixed order.
#include <hip/hip_runtime.h>

#include "pp_common.h"

namespace pp {

constexpr int32_t kTcSlice = 256;  // edges per slice
constexpr int32_t kTcLight = 16;   // lane-serial intersections up to this shorter row
// Owner rows up to kTcMid entries are searched in LDS by one wavefront (their
// tests are under 1% of the total on skewed graphs, and a bitmap costs the
// workgroup three barriers); longer ones become a bitmap, where bitmaps are large
// (kTcWide bytes) only those of more than kTcMidWide.
constexpr int32_t kTcMid = 64;
constexpr int32_t kTcMidWide = 512;
constexpr size_t kTcWide = 24576, kTcWidest = 65536;
// Lanes that stream one shorter row, and loads each keeps in flight.  R-MAT 16
// / 18, a call: 16 x 4 0.446 / 2.50 ms, 16 x 8 0.389 / 2.04, 32 x 4 0.380 /
// 2.20, 32 x 8 0.351 / 1.86, 64 x 4 0.402 / 2.22, 8 x 4 0.523 / 3.06.
constexpr int kTcGroup = 32;
constexpr int kTcLoads = 8;
constexpr int32_t kTcWindow = 1 << 20;      // vertices one bitmap covers (128 KB of LDS)
constexpr int32_t kTcMaxWaves = 16;

struct TcArgs {
    int32_t n;
    int64_t nnz;
    int32_t slices;
    const int32_t* off;  // caller's CSR (rows sorted ascending)
    const int32_t* idx;
    const int32_t* row;  // the row of every slot, where registration left it (nullable)
    int64_t* tc;         // [n] output (push: accumulator)
    int64_t* head;       // [slices] first segment of each slice (pull); before, edges of bitmap rows
    int64_t* tail;       // [slices] last segment of each slice (pull)
    int32_t* cnt;        // [nnz] |N(v) ∩ N(w)| of every slot; -1: not formed (NULL: none is)
    int32_t window;      // vertices per bitmap window
    int32_t* flag;       // bit 0: a row is not strictly ascending
};

// Index of the row holding edge j: largest v in [lo, hi) with off[v] <= j.
__device__ __forceinline__ int32_t row_of(const int32_t* off, int32_t lo, int32_t hi, int64_t j) {
    while (hi - lo > 1) {
        const int32_t mid = lo + (hi - lo) / 2;
        if (off[mid] <= j) lo = mid;
        else hi = mid;
    }
    return lo;
}

// |idx[a0, a1) ∩ idx[b0, b1)| for ascending rows, in one lane: every entry of
// the shorter row is searched in the longer one above the previous match.
__device__ __forceinline__ int64_t isect_lane(const int32_t* idx, int32_t a0, int32_t a1, int32_t b0, int32_t b1) {
    if (a1 - a0 > b1 - b0) {
        int32_t t = a0; a0 = b0; b0 = t;
        t = a1; a1 = b1; b1 = t;
    }
    int64_t cnt = 0;
    int32_t lo = b0;
    for (int32_t i = a0; i < a1 && lo < b1; ++i) {
        const int32_t x = idx[i];
        int32_t hi = b1;
        while (lo < hi) {
            const int32_t mid = lo + (hi - lo) / 2;
            if (idx[mid] < x) lo = mid + 1;
            else hi = mid;
        }
        if (lo < b1 && idx[lo] == x) {
            ++cnt;
            ++lo;
        }
    }
    return cnt;
}

// The same count by the whole wavefront (a0..b1 wave-uniform).  Lane l takes
// the l-th piece of the shorter row, finds its first entry's place in the
// longer row by binary search and merges forward.
__device__ __forceinline__ int64_t isect_wave(const int32_t* idx, int32_t a0, int32_t a1, int32_t b0, int32_t b1,
                                              int lane) {
    if (a1 - a0 > b1 - b0) {
        int32_t t = a0; a0 = b0; b0 = t;
        t = a1; a1 = b1; b1 = t;
    }
    const int32_t len = a1 - a0;
    const int32_t per = (len + kWave - 1) / kWave;
    const int32_t p0 = a0 + min(len, lane * per), p1 = a0 + min(len, (lane + 1) * per);
    int64_t cnt = 0;
    if (p0 < p1) {
        const int32_t x0 = idx[p0];
        int32_t lo = b0, hi = b1;
        while (lo < hi) {
            const int32_t mid = lo + (hi - lo) / 2;
            if (idx[mid] < x0) lo = mid + 1;
            else hi = mid;
        }
        int32_t i = p0;
        while (i < p1 && lo < b1) {
            const int32_t x = idx[i], y = idx[lo];
            if (x < y) ++i;
            else if (x > y) ++lo;
            else {
                ++cnt;
                ++i;
                ++lo;
            }
        }
    }
#pragma unroll
    for (int s = 32; s > 0; s >>= 1) cnt += __shfl_xor(cnt, s);
    return cnt;
}

// An edge of the slice, in LDS.
struct TcEdge {
    int32_t v, w;
    int32_t cnt;   // matches so far
    int32_t back;  // slot of the reverse edge, -1: not met
};

// Whether w's row is the one streamed when v and w meet: the owner has the
// longer row, equal rows go to the larger id.
__device__ __forceinline__ bool tc_owned(int32_t dv, int32_t v, int32_t dw, int32_t w) {
    return dw < dv || (dw == dv && w < v);
}

// One group of kTcGroup lanes streams the row piece [b, e) of edge k's w and
// adds the entries that `hit` accepts to the edge.
template <typename F>
__device__ __forceinline__ void tc_stream(const int32_t* idx, TcEdge& ed, int32_t b, int32_t e, int gl, F hit) {
    constexpr int U = kTcLoads;
    int32_t cnt = 0, back = -1;
    const int32_t v = ed.v;
    const int32_t* p = idx + b + gl;  // `left` slots from here to the row's end
    for (int32_t left = e - b - gl; left > 0; left -= U * kTcGroup, p += U * kTcGroup) {
        int32_t x[U];
#pragma unroll
        for (int k = 0; k < U; ++k) x[k] = p[min(k * kTcGroup, left - 1)];
#pragma unroll
        for (int k = 0; k < U; ++k) {
            if (k * kTcGroup < left) {
                cnt += hit(x[k]);
                if (x[k] == v) back = e - left + k * kTcGroup;
            }
        }
    }
#pragma unroll
    for (int s = kTcGroup / 2; s > 0; s >>= 1) cnt += __shfl_xor(cnt, s);
    if (gl == 0) ed.cnt += cnt;
    if (back >= 0) ed.back = back;
}

// First index in the ascending row piece [b, e) whose entry is >= x.
__device__ __forceinline__ int32_t tc_lower(const int32_t* idx, int32_t b, int32_t e, int32_t x) {
    while (b < e) {
        const int32_t mid = b + (e - b) / 2;
        if (idx[mid] < x) b = mid + 1;
        else e = mid;
    }
    return b;
}

// The pairs of a slice whose longer row has more than kTcLight entries, counted at
// the slot of the owner.  The slice's owned edges are compacted in slot order, rows
// with a bitmap first to s_list from the front, the others from the back, so a
// row's edges are consecutive.
//
// BITS: rows of more than CAP entries, by bitmap.  SEARCH: the others, searched in
// LDS.  Where the bitmap is small one launch does both.  Where it would leave a
// compute unit one workgroup or two, the searched rows have a launch of their own,
// of small workgroups and no bitmap, which also notes (in head) the slices that
// have rows for a bitmap; most sparse graphs have none.  One launch with a bitmap
// for every graph, against this: 1000 x 1031 grid 504 -> 136 us, ER n = 1M of degree
// 16 6.8 -> 1.9 ms, of 48 28.8 -> 6.7, n = 2.2M of 80 189 -> 36, a grid with a hub of
// 5,000 504 -> 156 us, R-MAT 20 (edge factor 8) 6.2 -> 5.9 ms.
template <int CAP, bool SEARCH, bool BITS>
__global__ __launch_bounds__(64 * (BITS ? kTcMaxWaves : 4)) void k_tc_count(TcArgs a) {
    constexpr int kWavesMax = BITS ? kTcMaxWaves : 4;
    extern __shared__ uint32_t bits[];  // BITS: window / 32 words
    __shared__ TcEdge s_edge[kTcSlice];
    __shared__ int16_t s_list[kTcSlice];     // owned edges, rows with a bitmap, then the searched ones
    __shared__ int16_t s_run[kTcSlice + 1];  // first list entry of every row
    __shared__ int32_t s_wbig[kTcSlice / kWave], s_wmid[kTcSlice / kWave], s_wrun[kTcSlice / kWave];
    __shared__ int32_t s_row[SEARCH ? kWavesMax : 1][SEARCH ? CAP : 1];
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wv = tid / kWave, nw = blockDim.x / kWave;
    const int grp = tid / kTcGroup, ngrp = blockDim.x / kTcGroup, gl = tid & (kTcGroup - 1);
    const uint64_t below = (1ull << lane) - 1ull;
    if (BITS)
        for (int32_t i = tid; i < a.window / 32; i += blockDim.x) bits[i] = 0u;
    for (int32_t s = blockIdx.x; s < a.slices; s += gridDim.x) {
        if (!SEARCH && a.head[s] == 0) continue;
        const int64_t e0 = (int64_t)s * kTcSlice;
        const int32_t ne = (int32_t)min((int64_t)kTcSlice, a.nnz - e0);
        __syncthreads();  // the lists of the previous slice are done with
        bool big = false, mid = false;
        if (tid < kTcSlice) {
            if (tid < ne) {
                const int32_t v = a.row ? a.row[e0 + tid] : row_of(a.off, 0, a.n, e0 + tid);
                const int32_t w = a.idx[e0 + tid];
                const int32_t dv = a.off[v + 1] - a.off[v], dw = a.off[w + 1] - a.off[w];
                if (dv > kTcLight && tc_owned(dv, v, dw, w)) {
                    big = dv > CAP;
                    mid = SEARCH && !big;
                } else if (SEARCH && BITS && max(dv, dw) <= kTcLight) {
                    // (few on the dense graphs of this form; k_tc_slices, which
                    // takes them otherwise, has a wavefront a slice)
                    a.cnt[e0 + tid] = (int32_t)isect_lane(a.idx, a.off[v], a.off[v + 1], a.off[w], a.off[w + 1]);
                }
                s_edge[tid] = TcEdge{v, w, 0, -1};
            }
        }
        const uint64_t mb = __ballot(big), mm = __ballot(mid);
        if (tid < kTcSlice && lane == 0) {
            s_wbig[wv] = __popcll(mb);
            s_wmid[wv] = __popcll(mm);
        }
        __syncthreads();
        int32_t nbig = 0, nmid = 0, pb = 0, pm = 0;
#pragma unroll
        for (int i = 0; i < kTcSlice / kWave; ++i) {
            if (i < wv) {
                pb += s_wbig[i];
                pm += s_wmid[i];
            }
            nbig += s_wbig[i];
            nmid += s_wmid[i];
        }
        if (!BITS) {
            if (tid == 0) a.head[s] = nbig;
            nbig = 0;
            big = false;
        }
        const int32_t nl = nbig + nmid;
        if (nl == 0) continue;
        if (big) s_list[pb + __popcll(mb & below)] = (int16_t)tid;
        if (mid) s_list[nbig + pm + __popcll(mm & below)] = (int16_t)tid;
        __syncthreads();
        // row starts in the list
        bool start = false;
        if (tid < nl) start = tid == 0 || tid == nbig || s_edge[s_list[tid]].v != s_edge[s_list[tid - 1]].v;
        const uint64_t ms = __ballot(start);
        if (tid < kTcSlice && lane == 0) s_wrun[wv] = __popcll(ms);
        __syncthreads();
        int32_t nrun = 0, pr = 0;
#pragma unroll
        for (int i = 0; i < kTcSlice / kWave; ++i) {
            if (i < wv) pr += s_wrun[i];
            nrun += s_wrun[i];
        }
        if (start) s_run[pr + __popcll(ms & below)] = (int16_t)tid;
        if (tid == 0) s_run[nrun] = (int16_t)nl;
        __syncthreads();
        // rows with a bitmap: the workgroup takes one after another
        int32_t r = 0;
        if constexpr (BITS) {
            for (; r < nrun && s_run[r] < nbig; ++r) {
                const int32_t k0 = s_run[r], k1 = s_run[r + 1];
                const int32_t ov = s_edge[s_list[k0]].v;
                const int32_t rb = a.off[ov], re = a.off[ov + 1];
                for (uint32_t lo = 0; lo < (uint32_t)a.n; lo += a.window) {
                    for (slot_t j = (slot_t)rb + tid; j < (slot_t)re; j += blockDim.x) {
                        const uint32_t p = (uint32_t)(a.idx[j] - lo);
                        if (p < (uint32_t)a.window) atomicOr(&bits[p >> 5], 1u << (p & 31));
                    }
                    __syncthreads();
                    for (int32_t k = k0 + grp; k < k1; k += ngrp) {
                        TcEdge& ed = s_edge[s_list[k]];
                        int32_t b = a.off[ed.w], e = a.off[ed.w + 1];
                        if (a.n > a.window) {
                            b = tc_lower(a.idx, b, e, (int32_t)lo);
                            e = (a.n - lo > (uint32_t)a.window) ? tc_lower(a.idx, b, e, (int32_t)lo + a.window) : e;
                        }
                        tc_stream(a.idx, ed, b, e, gl, [&](int32_t x) -> int32_t {
                            const uint32_t p = min((uint32_t)(x - lo), (uint32_t)a.window - 1u);
                            return (bits[p >> 5] >> (p & 31)) & 1u;
                        });
                    }
                    __syncthreads();
                    for (slot_t j = (slot_t)rb + tid; j < (slot_t)re; j += blockDim.x) {
                        const uint32_t p = (uint32_t)(a.idx[j] - lo);
                        if (p < (uint32_t)a.window) bits[p >> 5] = 0u;
                    }
                    __syncthreads();
                }
            }
        }
        // the other rows: one wavefront each, the row searched in LDS
        if constexpr (SEARCH) {
            for (r += wv; r < nrun; r += nw) {
                const int32_t k0 = s_run[r], k1 = s_run[r + 1];
                const int32_t ov = s_edge[s_list[k0]].v;
                const int32_t rb = a.off[ov], d = a.off[ov + 1] - rb;  // d <= CAP
                int32_t size = kWave;  // what is searched: the row, filled up to a power of two
                while (size < d) size <<= 1;
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                for (int32_t i = lane; i < size; i += kWave) s_row[wv][i] = i < d ? a.idx[rb + i] : INT32_MAX;
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                __builtin_amdgcn_wave_barrier();
                const int32_t* row = s_row[wv];
                for (int32_t k = k0 + lane / kTcGroup; k < k1; k += kWave / kTcGroup) {
                    TcEdge& ed = s_edge[s_list[k]];
                    tc_stream(a.idx, ed, a.off[ed.w], a.off[ed.w + 1], gl, [&](int32_t x) -> int32_t {
                        int32_t p = 0;  // largest p with row[p] <= x, or 0
                        if (CAP == kWave) {
#pragma unroll
                            for (int st = kWave / 2; st > 0; st >>= 1)
                                if (row[p + st] <= x) p += st;
                        } else {
                            for (int32_t st = size >> 1; st > 0; st >>= 1)
                                if (row[p + st] <= x) p += st;
                        }
                        return row[p] == x;
                    });
                }
                __builtin_amdgcn_wave_barrier();
            }
        }
        __syncthreads();
        if (tid < nl) {
            const int32_t k = s_list[tid];
            const TcEdge ed = s_edge[k];
            a.cnt[e0 + k] = ed.cnt;
            if (ed.back >= 0) a.cnt[ed.back] = ed.cnt;
        }
    }
}

// (eight wavefronts a SIMD: what it waits for is gathers)
template <bool PUSH>
__global__ __launch_bounds__(kBlock, 8) void k_tc_slices(TcArgs a) {
    const int lane = threadIdx.x & (kWave - 1);
    const int32_t gwave = blockIdx.x * (kBlock / kWave) + threadIdx.x / kWave;
    const int32_t nwaves = gridDim.x * (kBlock / kWave);
    for (int32_t s = gwave; s < a.slices; s += nwaves) {
        const int64_t e0 = (int64_t)s * kTcSlice;
        const int64_t e1 = min(e0 + kTcSlice, a.nnz);
        // rows holding the first and last edge of the slice bound every search
        int32_t v0 = 0, v1 = 0;
        if (!a.row) {
            if (lane == 0) v0 = row_of(a.off, 0, a.n, e0);
            if (lane == 1) v1 = row_of(a.off, 0, a.n, e1 - 1);
            v0 = __shfl(v0, 0);
            v1 = __shfl(v1, 1);
        }
        int64_t carry = 0;  // running sum of the open segment (row carry_v)
        int32_t carry_v = -1;
        for (int64_t jb = e0; jb < e1; jb += kWave) {
            const int64_t j = jb + lane;
            const bool live = j < e1;
            int32_t v = -1, w = -1, rb = 0, re = 0;
            int64_t cnt = 0;
            bool heavy = false;
            if (live) {
                v = a.row ? __builtin_nontemporal_load(a.row + j) : row_of(a.off, v0, v1 + 1, j);
                w = a.idx[j];
                rb = a.off[v];
                re = a.off[v + 1];
                cnt = a.cnt ? a.cnt[j] : -1;
                if (j + 1 < re && a.idx[j + 1] <= w) atomicOr(a.flag, 1);
                if (cnt < 0) {  // two short rows, a self-loop, or a one-way edge into a longer row
                    const int32_t wb = a.off[w], we = a.off[w + 1];
                    heavy = min(re - rb, we - wb) > kTcLight;
                    if (!heavy) cnt = isect_lane(a.idx, rb, re, wb, we);
                }
            }
            uint64_t hm = __ballot(heavy);
            while (hm) {
                const int src = __ffsll((long long)hm) - 1;
                hm &= hm - 1;
                const int32_t hv_b = __shfl(rb, src), hv_e = __shfl(re, src);
                const int32_t hw = __shfl(w, src);
                const int64_t c = isect_wave(a.idx, hv_b, hv_e, a.off[hw], a.off[hw + 1], lane);
                if (lane == src) cnt = c;
            }
            if (PUSH) {
                if (live && cnt) atomicAdd(reinterpret_cast<unsigned long long*>(&a.tc[w]), (unsigned long long)cnt);
                continue;
            }
            // pull: segmented inclusive sum over lanes of the same row (the
            // open segment of the previous round enters through lane 0)
            if (lane == 0 && v == carry_v) cnt += carry;
#pragma unroll
            for (int d = 1; d < kWave; d <<= 1) {
                const int64_t y = __shfl_up(cnt, d);
                const int32_t yv = __shfl_up(v, d);
                if (lane >= d && yv == v) cnt += y;
            }
            // a segment ends where its row or the slice ends; one that reaches
            // lane 63 otherwise stays open into the next round
            const bool seg_end = live && (j + 1 >= e1 || j + 1 >= re);
            if (seg_end) {
                const bool starts_here = rb >= e0, ends_here = re <= e1;
                if (starts_here && ends_here) {
                    a.tc[v] = cnt / 2;
                } else {
                    if (!starts_here) a.head[s] = cnt;  // the slice's first segment
                    if (!ends_here) a.tail[s] = cnt;    // the slice's last segment
                }
            }
            const int src = min(kWave - 1, (int)(e1 - 1 - jb));
            carry = __shfl(cnt, src);
            carry_v = __shfl(v, src);
        }
    }
}

// Pull: counters of rows that cross slices, and of empty rows.
__global__ __launch_bounds__(kBlock) void k_tc_fix(TcArgs a) {
    const int lane = threadIdx.x & (kWave - 1);
    const int32_t t = blockIdx.x * blockDim.x + threadIdx.x;
    const int32_t stride = gridDim.x * blockDim.x;
    for (int32_t base = t - lane; base < a.n; base += stride) {
        const int32_t v = base + lane;
        int64_t rb = 0, re = 0;
        if (v < a.n) {
            rb = a.off[v];
            re = a.off[v + 1];
        }
        const int32_t s0 = (int32_t)(rb / kTcSlice), s1 = (int32_t)((re - 1) / kTcSlice);
        const bool span = v < a.n && re > rb && s1 > s0;
        if (v < a.n && re == rb) a.tc[v] = 0;
        // short spans in the lane, long ones (hub rows) by the wavefront
        const bool longspan = span && (s1 - s0) > 8;
        if (span && !longspan) {
            int64_t sum = a.tail[s0];
            for (int32_t s = s0 + 1; s <= s1; ++s) sum += a.head[s];
            a.tc[v] = sum / 2;
        }
        uint64_t lm = __ballot(longspan);
        while (lm) {
            const int src = __ffsll((long long)lm) - 1;
            lm &= lm - 1;
            const int32_t b = __shfl(s0, src), e = __shfl(s1, src);
            int64_t sum = 0;
            for (int32_t s = b + 1 + lane; s <= e; s += kWave) sum += a.head[s];
#pragma unroll
            for (int d = 32; d > 0; d >>= 1) sum += __shfl_xor(sum, d);
            if (lane == src) a.tc[v] = (sum + a.tail[b]) / 2;
        }
    }
}

// Counters to zero, slot counts to "not formed".
__global__ void k_tc_zero(TcArgs a) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t v = t; v < a.n; v += stride) a.tc[v] = 0;
    for (int64_t j = t; a.cnt && j < a.nnz; j += stride) a.cnt[j] = -1;
    if (blockIdx.x == 0 && threadIdx.x == 0) *a.flag = 0;
}

__global__ void k_tc_halve(int32_t n, int64_t* tc) {
    for (int32_t v = blockIdx.x * blockDim.x + threadIdx.x; v < n; v += gridDim.x * blockDim.x) tc[v] /= 2;
}

struct TcLayout {
    size_t flag, head, tail, cnt, total;
    int32_t slices;
};

static TcLayout tc_layout(int64_t nnz) {
    TcLayout L{};
    L.slices = (int32_t)((nnz + kTcSlice - 1) / kTcSlice);
    size_t p = 0;
    auto take = [&](size_t bytes) {
        size_t at = p;
        p = align_up(p + bytes, 256);
        return at;
    };
    L.flag = take(sizeof(int32_t));
    L.head = take((size_t)std::max(L.slices, 1) * 8);
    L.tail = take((size_t)std::max(L.slices, 1) * 8);
    L.cnt = take((size_t)std::max<int64_t>(nnz, 1) * 4);
    L.total = p;
    return L;
}

// Threads of a counting workgroup: as many as keep a compute unit's
// wavefronts busy beside the LDS its bitmap takes (160 KB: 8 x 8 KB bitmaps
// at 65,536 vertices, one of 128 KB from a million).
static int32_t tc_threads(size_t bitmap_bytes) {
    return bitmap_bytes <= 24576 ? 256 : bitmap_bytes <= 65536 ? 512 : 1024;
}

}  // namespace pp

using namespace pp;

PP_EXPORT size_t pp_tc_workspace_bytes(pp_graph g) { return g ? tc_layout(g->d.nnz).total : 0; }

PP_EXPORT pp_status pp_tc_run(pp_graph g, pp_dir dir, int64_t* tc, void* ws, size_t ws_bytes, void* stream) {
    clear_error();
    if (!g) return set_error(PP_E_NULL, "graph handle is NULL");
    if (!tc || !ws) return set_error(PP_E_NULL, "tc and ws are required");
    if (dir != PP_PUSH && dir != PP_PULL) return set_error(PP_E_RANGE, "dir must be PP_PUSH or PP_PULL");
    const TcLayout L = tc_layout(g->d.nnz);
    if (ws_bytes < L.total) return set_error(PP_E_WORKSPACE, "TC workspace too small");
    if (reinterpret_cast<uintptr_t>(ws) % 256 != 0) return set_error(PP_E_RANGE, "ws must be 256-byte aligned");
    char* w = static_cast<char*>(ws);
    TcArgs a;
    a.n = g->d.n;
    a.nnz = g->d.nnz;
    a.slices = L.slices;
    a.off = g->d.user_csr_off;
    a.idx = g->d.user_csr_idx;
    a.tc = tc;
    a.head = reinterpret_cast<int64_t*>(w + L.head);
    a.tail = reinterpret_cast<int64_t*>(w + L.tail);
    a.flag = reinterpret_cast<int32_t*>(w + L.flag);
    // no counts beforehand: rows of at most kTcLight entries, or hardly longer ones
    // in a sparse graph, where looking for the pairs costs more than they do (ER
    // n = 2M of degree 4: 750 us looked for, 570 without)
    const int32_t longest = g->max_out_deg;
    const bool sparse = longest <= kTcLight || (longest <= kTcMid && a.nnz < 8 * (int64_t)a.n);
    // few slices leave most of the chip idle: what counts then is that a slice has a
    // workgroup instead of the wavefront of k_tc_slices, and one launch does it all
    // (ER, degree x n, us a call without / with: 4 x 5,591 60 / 46, 8 x 5,591 76 / 60,
    // 16 x 20,001 117 / 89, 4 x 80,001 68 / 59; level at 8 x 45,001 and 12 x 65,535)
    a.window = (int32_t)std::min<int64_t>(((int64_t)a.n + 63) / 64 * 64, kTcWindow);
    const size_t lds = (size_t)a.window / 8;
    const bool few = lds <= kTcWide && a.slices <= (sparse ? 5 : 12) * g->num_cu;
    const bool count = few || !sparse;
    a.cnt = count ? reinterpret_cast<int32_t*>(w + L.cnt) : nullptr;
    // (k_tc_slices alone is as well off with its bounded search: grids 25% faster by
    // the list, sparse ER 10% slower)
    a.row = count && !g->relabelled && g->d.aliased ? g->d.csc_row : nullptr;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const int32_t vb = std::max(1, std::min(ceil_div(a.n, kBlock), 4096));
    const int32_t zb = std::max(1, std::min(ceil_div(std::max<int64_t>(a.n, a.nnz), kBlock), 4096));
    hipLaunchKernelGGL(k_tc_zero, dim3(zb), dim3(kBlock), 0, st, a);
    if (a.slices > 0) {
        // (a bitmap of kTcWidest bytes leaves a compute unit two workgroups, which
        // still is the better form where most pairs need one: R-MAT 18 1.7 ms, 2.3 in
        // two launches; ER n = 300,000 of degree 40 needs none: 2.6 -> 1.6 ms)
        auto search = [&](auto kern) {
            hipLaunchKernelGGL(kern, dim3(std::min(a.slices, g->num_cu * 64)), dim3(4 * kWave), 0, st, a);
        };
        auto with_bits = [&](auto kern) {
            allow_dynamic_lds(reinterpret_cast<const void*>(kern), lds);
            // a workgroup clears its bitmap once: few workgroups where that is long
            const int32_t wgs = g->num_cu * 16 * (1024 / tc_threads(lds));
            hipLaunchKernelGGL(kern, dim3(std::min(a.slices, wgs)), dim3(tc_threads(lds)), lds, st, a);
        };
        if (!count) {
            // k_tc_slices alone
        } else if (longest <= kTcMid && !few) {
            search(&k_tc_count<kTcMid, true, false>);
        } else if (lds <= kTcWide || (lds <= kTcWidest && longest > kTcMidWide && a.nnz >= 8 * (int64_t)a.n)) {
            with_bits(&k_tc_count<kTcMid, true, true>);
        } else {
            search(&k_tc_count<kTcMidWide, true, false>);
            if (longest > kTcMidWide) with_bits(&k_tc_count<kTcMidWide, false, true>);
        }
        const int32_t blocks = std::min(ceil_div(a.slices, kBlock / kWave), g->num_cu * 8);
        if (dir == PP_PUSH) hipLaunchKernelGGL(k_tc_slices<true>, dim3(blocks), dim3(kBlock), 0, st, a);
        else hipLaunchKernelGGL(k_tc_slices<false>, dim3(blocks), dim3(kBlock), 0, st, a);
    }
    if (dir == PP_PUSH) hipLaunchKernelGGL(k_tc_halve, dim3(vb), dim3(kBlock), 0, st, a.n, a.tc);
    else hipLaunchKernelGGL(k_tc_fix, dim3(vb), dim3(kBlock), 0, st, a);
    PP_LAUNCH_CHECK("k_tc_slices");
    int32_t flag = 0;
    PP_HIP(hipMemcpyAsync(&flag, a.flag, sizeof(int32_t), hipMemcpyDeviceToHost, st));
    PP_HIP(hipStreamSynchronize(st));
    if (flag) return set_error(PP_E_GRAPH, "triangle counting needs rows in strictly ascending order");
    return PP_OK;
}
