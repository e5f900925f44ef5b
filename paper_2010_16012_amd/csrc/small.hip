// PageRank of a small graph in one launch (Sec. 3.1 equation, Jacobi steps): a
// workgroup keeps the whole graph -- the in-edges in registers, the vectors in
// LDS -- and runs every step itself.
//
// A step of a thousand vertices is a few microseconds of work on one compute
// unit and a kernel launch takes 5, so launched step by step it is the launches
// that are paid for.  Here the rows are cut into pieces of kSmallPiece slots
// (the last one padded), a thread holds Q consecutive pieces, and a step is:
// sum every piece (one LDS read a slot, no branches), close the rows that end
// inside the thread, scan the open ends across the workgroup, close the rest;
// two barriers.  Whoever closes a row writes its next contribution into the
// other of two vectors.  Fixed summation order: bit-reproducible, both forms
// alike (inside one workgroup nothing is shared that a form could contend for).
#include <hip/hip_runtime.h>

#include "pp_common.h"
#include "sweep.h"

namespace pp {

constexpr int kSmallPiece = 4;
constexpr int kSmallMaxWaves = 16;

struct SmallArgs {
    int32_t n, iters;
    const int32_t* off;    // CSC
    const int32_t* idx;
    const float* wt;       // weights in CSC slot order (weighted only)
    const float* inv_s;
    const int32_t* perm;
    const float* x;        // x_0 in caller ids; NULL: the unit vector of tele_v
    float* y;              // x_iters, y[caller id * y_stride]
    int64_t y_stride;
    float base, tele, f;
    int32_t tele_v;
};

// The new rank of row r from its gathered sum: the next contribution, or (after
// the last step) the output.
__device__ __forceinline__ void small_finish(const SmallArgs& a, const float* inv, float* nxt, bool last, int32_t r,
                                             float acc) {
    const float yv = a.base + ((r == a.tele_v) ? a.tele : 0.f) + acc;
    if (last) a.y[(int64_t)user_id(a.perm, r) * a.y_stride] = yv;
    else nxt[r] = a.f * yv * inv[r];
}

template <int Q, bool W>
__global__ __launch_bounds__(64 * kSmallMaxWaves) void k_pr_small(SmallArgs a) {
    constexpr int P = kSmallPiece;
    extern __shared__ float lds[];
    const int32_t n = a.n;
    float* cur = lds;                // contributions, and a zero for padding slots
    float* nxt = cur + n + 1;
    float* inv = nxt + n + 1;
    uint16_t* pre = reinterpret_cast<uint16_t*>(inv + n);  // [n + 1] first piece of a row
    __shared__ float s_open[kSmallMaxWaves];
    __shared__ int32_t s_fresh[kSmallMaxWaves];
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wv = tid / kWave;
    const int T = blockDim.x, nw = T / kWave;
    for (int32_t r = tid; r < n; r += T) {
        const float is = a.inv_s[r];
        const float x0 = a.x ? a.x[user_id(a.perm, r)] : (r == a.tele_v ? 1.f : 0.f);
        inv[r] = is;
        cur[r] = a.f * x0 * is;
    }
    if (tid == 0) cur[n] = nxt[n] = 0.f;
    // first pieces: every thread a run of rows
    const int32_t per = (n + T - 1) / T, r0 = min(n, tid * per), r1 = min(n, r0 + per);
    int32_t mine = 0;
    for (int32_t r = r0; r < r1; ++r) mine += (a.off[r + 1] - a.off[r] + P - 1) / P;
    const int incl = wave_incl_sum(mine);
    if (lane == kWave - 1) s_fresh[wv] = incl;
    __syncthreads();
    int32_t at = incl - mine, total = 0;
    for (int q = 0; q < nw; ++q) {
        if (q < wv) at += s_fresh[q];
        total += s_fresh[q];
    }
    for (int32_t r = r0; r < r1; ++r) {
        pre[r] = (uint16_t)at;
        at += (a.off[r + 1] - a.off[r] + P - 1) / P;
    }
    if (tid == 0) pre[n] = (uint16_t)total;
    __syncthreads();
    // this thread's pieces: LDS byte offsets of their sources, two to a
    // register; rows; which of them begin a row
    uint32_t src[Q * P / 2];
    float wt[W ? Q * P : 1];
    int32_t row[Q];
    uint32_t heads = 0;
    {
        const int32_t p0 = tid * Q;
        int32_t lo = 0, hi = n;  // the last row with pre[row] <= p0
        while (hi - lo > 1) {
            const int32_t mid = (lo + hi) >> 1;
            if ((int32_t)pre[mid] <= p0) lo = mid;
            else hi = mid;
        }
        int32_t r = lo;
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const int32_t p = p0 + q;
            int32_t b = 0, e = 0;
            if (p < total) {
                while (p >= (int32_t)pre[r + 1]) ++r;
                b = a.off[r] + (p - pre[r]) * P;
                e = a.off[r + 1];
                if (p == (int32_t)pre[r]) heads |= 1u << q;
            }
            row[q] = r;
#pragma unroll
            for (int k = 0; k < P; ++k) {
                const uint32_t o = (uint32_t)(b + k < e ? a.idx[b + k] : n) * 4u;
                if (W) wt[q * P + k] = b + k < e ? a.wt[b + k] : 0.f;
                const int i = q * P + k;
                src[i / 2] = (i & 1) ? (src[i / 2] | (o << 16)) : o;
            }
        }
    }
    const bool any = heads != 0;
    // the row open where this thread starts: closed here if a row begins here
    const int32_t row_before = (tid * Q > 0 && tid * Q <= total) ? ([&] {
        int32_t r = row[0];
        if (heads & 1u) {  // the last non-empty row before row[0]
            do --r;
            while (pre[r] == pre[r + 1]);
        }
        return r;
    })() : -1;
    const bool ends = tid * Q < total && tid * Q + Q >= total;  // holds the last piece
    const int32_t row_last = row[Q - 1];
    for (int32_t it = 0; it < a.iters; ++it) {
        const bool last = it == a.iters - 1;
        const char* cb = reinterpret_cast<const char*>(cur);
        float s[Q];
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            float v[P];
#pragma unroll
            for (int k = 0; k < P; ++k) {
                const int i = q * P + k;
                // unpacked anew in every step: kept unpacked they would fill
                // the registers
                if (!(i & 1)) asm volatile("" : "+v"(src[i / 2]));
                const uint32_t o = (i & 1) ? src[i / 2] >> 16 : src[i / 2] & 0xFFFFu;
                v[k] = *reinterpret_cast<const float*>(cb + o);
                if (W) v[k] *= wt[i];
            }
            s[q] = (v[0] + v[1]) + (v[2] + v[3]);
        }
        float run = 0.f, lead = 0.f;
        bool first = true;
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            if (heads & (1u << q)) {
                if (first) lead = run;
                else small_finish(a, inv, nxt, last, row[q > 0 ? q - 1 : 0], run);
                run = 0.f;
                first = false;
            }
            run += s[q];
        }
        // what the row open at the end of each lane holds so far
        float open = run;
        int fresh = any ? 1 : 0;
        seg_step<0x111>(open, fresh);
        seg_step<0x112>(open, fresh);
        seg_step<0x114>(open, fresh);
        seg_step<0x118>(open, fresh);
        seg_step<0x142, 0xa>(open, fresh);
        seg_step<0x143, 0xc>(open, fresh);
        float before = dpp_takef<0x138>(open);  // ... at its start
        const int fresh_before = dpp_take<0x138>(fresh);
        if (lane == kWave - 1) {
            s_open[wv] = open;
            s_fresh[wv] = fresh;
        }
        __syncthreads();
        float carry = 0.f;
        for (int q = 0; q < wv; ++q) carry = s_fresh[q] ? s_open[q] : carry + s_open[q];
        if (!fresh_before) before = carry + before;
        if (any && row_before >= 0) small_finish(a, inv, nxt, last, row_before, before + lead);
        if (ends) small_finish(a, inv, nxt, last, row_last, fresh ? open : carry + open);
        // rows without in-edges: the same from the first step on
        if (it < 2 || last)
            for (int32_t r = tid; r < n; r += T)
                if (pre[r] == pre[r + 1]) small_finish(a, inv, nxt, last, r, 0.f);
        __syncthreads();
        float* t = cur;
        cur = nxt;
        nxt = t;
    }
}

// Graphs one workgroup takes: up to kSmallQ pieces a thread (a weighted graph
// keeps its weights in registers too) and kSmallN vertices.  20 steps, each
// call waited for, launched step by step -> here: R-MAT 8 125 -> 45 us, 9 139
// -> 55, 10 144 -> 74, ER n = 2,001 (20,000 edges) 167 -> 79; weighted R-MAT 10
// 135 -> 81.  At 12 pieces a thread the registers spill: 149 -> 114 at 48,000
// slots, and past 60,000 one compute unit is slower than the launches.
constexpr int32_t kSmallN = 10240;
constexpr int kSmallQ = 8, kSmallQW = 6;

template <int Q>
static void launch_small_q(const SmallArgs& a, bool weighted, int32_t threads, size_t lds, hipStream_t st) {
    if (weighted) {
        constexpr int QW = Q < kSmallQW ? Q : kSmallQW;  // small_for admits no more
        allow_dynamic_lds(reinterpret_cast<const void*>(&k_pr_small<QW, true>), lds);
        hipLaunchKernelGGL((k_pr_small<QW, true>), dim3(1), dim3(threads), lds, st, a);
    } else {
        allow_dynamic_lds(reinterpret_cast<const void*>(&k_pr_small<Q, false>), lds);
        hipLaunchKernelGGL((k_pr_small<Q, false>), dim3(1), dim3(threads), lds, st, a);
    }
}

// Pieces at most: every non-empty row pads its last one.
static int64_t small_pieces(pp_graph g) {
    const int64_t rows = std::min<int64_t>(g->d.n - g->empty_in, g->d.nnz);
    return (g->d.nnz + (kSmallPiece - 1) * rows) / kSmallPiece;
}

static size_t small_lds(int32_t n) { return (size_t)n * 14 + 16; }

// Pulls, and pushes whose updates may be buffered (pp_set_push_bins).
bool small_for(pp_graph g, pp_dir dir) {
    const GraphDev& d = g->d;
    if (d.n > kSmallN || d.nnz < 1 || small_lds(d.n) > (size_t)g->max_lds - 1024) return false;
    if (small_pieces(g) > (int64_t)kSmallMaxWaves * kWave * (g->weighted ? kSmallQW : kSmallQ)) return false;
    return dir == PP_PULL || (dir == PP_PUSH && g->tune.push_bins && g->tune.hot > 0 && g->transposed);
}

// All steps of a run: x_0 = x (caller ids; NULL: the unit vector of
// tp.vertex), iters >= 1 steps, the last iterate to y (may be x).
pp_status launch_small(pp_graph g, int32_t iters, float f, const float* x, float* y, const Teleport& tp,
                       hipStream_t st) {
    const GraphDev& d = g->d;
    SmallArgs a{};
    a.n = d.n;
    a.iters = iters;
    a.off = d.csc_off;
    a.idx = d.csc_idx;
    a.wt = d.csc_w;
    a.inv_s = d.inv_s;
    a.perm = d.perm;
    a.x = x;
    a.y = y;
    a.y_stride = tp.y_stride;
    a.base = tp.base;
    a.tele = tp.extra;
    a.tele_v = tp.vertex;
    a.f = f;
    const int64_t pieces = small_pieces(g);
    const int32_t threads = pieces <= 4 * 256 ? 256 : pieces <= 4 * 512 ? 512 : 1024;
    const int32_t q = ceil_div(pieces, threads);
    const size_t lds = small_lds(d.n);
    if (q <= 2) launch_small_q<2>(a, g->weighted, threads, lds, st);
    else if (q <= 4) launch_small_q<4>(a, g->weighted, threads, lds, st);
    else if (q <= 6) launch_small_q<6>(a, g->weighted, threads, lds, st);
    else launch_small_q<8>(a, g->weighted, threads, lds, st);
    PP_LAUNCH_CHECK("k_pr_small");
    return PP_OK;
}

}  // namespace pp
