// Kernels of the single-query launch (init, persistent solver, unpack).
// Kept apart from the host code in sssp.hip so that the device code the
// counter summaries were taken on can be identified by these files alone.
#pragma once
#include <hip/hip_runtime.h>
#include <limits.h>

#include "sssp_device.hpp"
#include "sssp_init.hpp"
#include "sssp_small.hpp"
#include "sssp_sweep.hpp"

namespace {

// ---------------------------------------------------------------------------
// init: keys, the per-block weight range, and (block 0) the control block
// with the source already enqueued
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(INIT_WG) void k_init(Queue q, long long* key, int n, int src,
                                                  unsigned shift, const int* w, long long m,
                                                  int* wrange /* [2 * gridDim.x] */) {
    const long long tid = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    const long long stride = (long long)gridDim.x * blockDim.x;
    init_keys(key, n, src, shift, tid, stride);
    int lo, hi;
    weight_range(w, m, tid, stride, lo, hi);
    block_weight_range(lo, hi, wrange);
    if (blockIdx.x != 0 || threadIdx.x != 0) return;
    bq::Ctrl* c = q.ctrl;
    c->pending.v = 1ull;
    c->abort.v = 0ull;
    c->error.v = 0ull;
    c->negcycle.v = 0ull;
    c->aux[0].v = (unsigned long long)gridDim.x;  // number of weight-range partials
    c->aux[1].v = (unsigned long long)LLONG_MIN;  // near / far threshold (buckets)
    c->busy.v = 0ull;
    for (unsigned sg = 0; sg < MAX_Q; ++sg)        // dequeue positions at start
        q.ctrl[sg].aux[2].v = q.ctrl[sg].head.v;
    c->aux[4].v = bq::now_ticks();                // clock at start
    c->aux[5].v = 0ull;                           // strips that solved the query
    for (int i = 0; i < bq::ST_N; ++i) c->stats[i].v = 0ull;
    // enqueue src: the queue is quiescent, so slot (tail mod N) is free for
    // this round (ticket 2r) and count is 0
    const unsigned long long pos = c->tail.v;
    const unsigned slot = (unsigned)(pos & (q.N - 1ull));
    const unsigned round = (unsigned)(pos >> q.logN);
    q.slots[slot] = bq::slot_word(2u * round + 1u, (unsigned)src);
    c->tail.v = pos + 1ull;
    c->count.v = 1ull;
}

template <int B, int UU>
__device__ __forceinline__ void solve_kernel_body(const SolveArgs& a) {
    if (solved_before(a)) {
        // take back the source that k_init has enqueued
        if (blockIdx.x == 0 && threadIdx.x == 0) {
            bq::Ctrl* c = (bq::Ctrl*)a.q.ctrl;
            const unsigned long long pos = c->tail.v - 1ull;
            a.q.slots[pos & (a.q.N - 1ull)] =
                bq::slot_word(2u * ((uint32_t)(pos >> a.q.logN) + 1u), 0u);
            c->head.v = pos + 1ull;
            c->count.v = 0ull;
            c->aux[5].v = *a.taken;
        }
        return;
    }
    __shared__ WaveLds<B> lds[WAVES_PER_WG_ONE];
    __shared__ WgShared S;
    WaveLds<B>& L = lds[threadIdx.x >> 6];
    const int wid = (int)(threadIdx.x >> 6);
    if (threadIdx.x == 0) {
        S.poller = -1;
        S.wake = 0u;
        S.done = 0;
    }
    __syncthreads();
    WaveStats st{};
    solve_instance<B, true, UU>(a, L, S, wid, st);
    flush_stats(a.q.ctrl->stats, st);
}

template <int B>
__global__ __launch_bounds__(SOLVE_WG_ONE, SSSP_MIN_WAVES) void k_solve(SolveArgs a) {
    solve_kernel_body<B, U>(a);
}

// the same solver with SHORT_ROW_UNROLL edges per lane per scan step, for
// graphs whose rows are short on average (see launch_solve)
template <int B, int UU>
__global__ __launch_bounds__(SOLVE_WG_ONE, SSSP_MIN_WAVES) void k_solve_short(SolveArgs a) {
    solve_kernel_body<B, UU>(a);
}

// k_init's work (keys, weight range, control words) for the sweep form: also
// notes the longest row, clears the stamps of rows longer than C, and puts the
// source into the first buffer.
__global__ __launch_bounds__(INIT_WG) void k_sweep_init(SolveArgs a, SweepArgs f, int* wrange) {
    const long long tid = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    const long long stride = (long long)gridDim.x * blockDim.x;
    const long long C = 1ll << a.chunk_log;
    init_keys((long long*)a.key, a.n, a.src, a.shift, tid, stride);
    int lo, hi;
    weight_range((const int*)a.w, a.m, tid, stride, lo, hi);
    long long lr = 0;
    for (long long v = tid; v < a.n; v += stride) {
        const long long deg = a.off[v + 1] - a.off[v];
        lr = deg > lr ? deg : lr;
        if (deg > C) f.stamp[v] = 0u;
    }
    if (f.p.ctl != nullptr) strip_seed(f.p, a.n, 0, a.n, true, tid, stride);
    __shared__ unsigned slr;
    if (threadIdx.x == 0) slr = 0u;
    block_weight_range(lo, hi, wrange);  // synchronizes
    note_row(&slr, lr);
    __syncthreads();
    if (threadIdx.x == 0) f.longp[blockIdx.x] = slr;
    if (blockIdx.x != 0) return;
    // block 0: control words and the source's items
    sweep_seed(a, f, threadIdx.x, INIT_WG);
    if (threadIdx.x != 0) return;
    BQ_GLOBAL bq::Ctrl* q = a.q.ctrl;
    q->abort.v = 0ull;
    q->error.v = 0ull;
    q->negcycle.v = 0ull;
    q->aux[0].v = (unsigned long long)gridDim.x;  // number of partials
    q->aux[4].v = bq::now_ticks();                // clock at start
    q->aux[5].v = 0ull;                           // strips that solved the query
    for (int i = 0; i < bq::ST_N; ++i) q->stats[i].v = 0ull;
}

__global__ __launch_bounds__(SWEEP_WG) void k_sweep(SolveArgs a, SweepArgs f) {
    __shared__ SweepLds<SWEEP_WAVES> S;
    if (solved_before(a)) {
        if (blockIdx.x == 0 && threadIdx.x == 0) a.q.ctrl->aux[5].v = *a.taken;
        return;
    }
    WaveStats st{};
    sweep_instance<SWEEP_WAVES>(a, f, gridDim.x, S, st);
    sum_stats(S.stats, st);
    if (threadIdx.x < (unsigned)bq::ST_N && S.stats[threadIdx.x])
        bq::add_rlx(&a.q.ctrl->stats[threadIdx.x].v, S.stats[threadIdx.x]);
}

// The words of a strip solve whose query falls to the asynchronous solver if
// the strip form refuses it, and the longest row.
__global__ __launch_bounds__(INIT_WG) void k_strip_init(StripArgs p, const long long* off, int n,
                                                        unsigned* longp) {
    const long long tid = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    const long long stride = (long long)gridDim.x * blockDim.x;
    strip_seed(p, n, 0, n, true, tid, stride);
    long long lr = 0;
    for (long long v = tid; v < n; v += stride)
        lr = off[v + 1] - off[v] > lr ? off[v + 1] - off[v] : lr;
    __shared__ unsigned slr;
    if (threadIdx.x == 0) slr = 0u;
    __syncthreads();
    note_row(&slr, lr);
    __syncthreads();
    if (threadIdx.x == 0) longp[blockIdx.x] = slr;
}

__global__ __launch_bounds__(STRIP_WG) void k_strip(SolveArgs a, StripArgs p) {
    extern __shared__ __align__(16) unsigned char lds[];
    StripLds& S = *(StripLds*)lds;
    WaveStats st{};
    strip_instance(a, p, S, st);
    sum_stats(S.stats, st);
    if (threadIdx.x < (unsigned)bq::ST_N && S.stats[threadIdx.x])
        bq::add_rlx(&a.q.ctrl->stats[threadIdx.x].v, S.stats[threadIdx.x]);
}

// One query on one workgroup. `h` is the host's copy of the control block
// (pinned memory): the result words and counters are stored there directly.
__global__ __launch_bounds__(SMALL_WG) void k_small(SolveArgs a, int* pred, bq::Ctrl* h) {
    extern __shared__ __align__(16) unsigned char lds[];
    // the CSR check of the same call comes before the solve in the stream, and
    // the host reads its word with the result (waiting for it first cost 20 us)
    const unsigned long long defects = a.taken != nullptr ? *a.taken : 0ull;
    if (threadIdx.x == 0) h->aux[3].v = defects;
    if (defects != 0ull) return;
    WaveStats st{};
    const SmallResult r = small_instance(a, (long long*)a.key, pred, nullptr, lds, st);
    SmallLds& S = *(SmallLds*)lds;
    sum_stats(S.stats, st);
    if (threadIdx.x < (unsigned)bq::ST_N) h->stats[threadIdx.x].v = S.stats[threadIdx.x];
    if (threadIdx.x != 0) return;
    h->error.v = (unsigned long long)r.err;
    h->negcycle.v = (unsigned long long)r.neg;
    h->abort.v = 0ull;
}

// dist[v] = d, pred[v] = parent (INT64_MAX / -1 when unreached; pred[src] = -1;
// INT64_MIN / -1 for minus infinity)
__global__ void k_unpack(long long* key, int* pred, int n, int src, unsigned shift) {
    const long long dmax = KEY_INF >> shift;
    const unsigned pmask = (1u << (shift - 1u)) - 1u;
    for (long long v = (long long)blockIdx.x * blockDim.x + threadIdx.x; v < n;
         v += (long long)gridDim.x * blockDim.x) {
        const long long k = key[v];
        if (is_neg_key(k)) {  // minus infinity (marking mode)
            key[v] = LLONG_MIN;
            if (pred) pred[v] = -1;
            continue;
        }
        const long long d = k >> shift;
        const bool reached = d != dmax;
        key[v] = reached ? d : LLONG_MAX;
        if (pred) pred[v] = (reached && v != src) ? (int)(((unsigned long long)k >> 1) & pmask) : -1;
    }
}

}  // namespace
