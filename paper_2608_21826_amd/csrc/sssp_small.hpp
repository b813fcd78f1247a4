// The queue-driven Bellman-Ford on one workgroup (Section III.C), for graphs
// whose keys and queue fit one CU's LDS.
//
// Same keys, relaxations and results as the other forms. The keys (8 B per
// vertex), the row starts (4 B) and both queue buffers (2 B per entry) live in
// LDS, so lowering a label, publishing and the meeting between sweeps cost LDS
// round trips and a workgroup barrier instead of memory-side atomics and a
// barrier over the chip (1.25 against 6.4 us per sweep on a 64 x 64 grid); the
// columns and weights are read through the caches. Weight range, solve and
// unpack are one launch.
//
// A sweep gives each item to G lanes, G the power of two at or above the
// average row length, SMALL_U items per group at a time. A row longer than
// SMALL_HUB * G is left for the next sweep, where all 16 waves scan it together.
#pragma once
#include <hip/hip_runtime.h>
#include <limits.h>

#include <type_traits>

#include "sssp_device.hpp"
#include "sssp_init.hpp"

namespace {

constexpr int SMALL_WG = 1024;
constexpr int SMALL_WAVES = SMALL_WG / 64;
constexpr int SMALL_U = 4;            // items per lane group in flight
constexpr int SMALL_HUB = 16;         // steps of G edges a row may take alone
constexpr unsigned SMALL_HUBS = 128;  // long rows left per sweep; more are scanned alone
constexpr unsigned SMALL_MAX_N = 9984;       // what the LDS holds
constexpr long long SMALL_MAX_M = 40960;      // but for meshes, see is_small in sssp.hip

struct SmallLds {
    long long red[SMALL_WAVES][2];
    unsigned cnt[3];        // items of a buffer, by sweep mod 3
    unsigned nhub[3];       // long rows left for a sweep
    unsigned hub[2][SMALL_HUBS];
    long long hub_d[2][SMALL_HUBS];  // their sources' packed labels
    unsigned long long stats[bq::ST_N];
    int neg, err;
    unsigned stop;          // 1 + the sweep that stopped the solve, 0 if none
};

// LDS bytes of a graph of n vertices
constexpr size_t small_lds_bytes(int n) {
    return ((sizeof(SmallLds) + 15) & ~(size_t)15) + 16u * (size_t)n + 32u;
}
constexpr size_t small_lds_bytes_max() { return small_lds_bytes((int)SMALL_MAX_N); }

struct SmallResult {
    int neg, err;
};

// What a solve reads of its SolveArgs: the CSR, n, m, src, shift, deadline,
// neginf. `dist` and `pred` (may be null) are its outputs; with `reached` the
// number of edges whose source vertex was reached is added to it. Whole
// workgroup; `st` is per wave as in the other forms.
__device__ SmallResult small_instance(const SolveArgs& a, long long* dist, int* pred,
                                      unsigned long long* reached, unsigned char* lds,
                                      WaveStats& st) {
    SmallLds& S = *(SmallLds*)lds;
    long long* key = (long long*)(lds + ((sizeof(SmallLds) + 15) & ~(size_t)15));
    unsigned* row = (unsigned*)(key + a.n);                    // [n + 1] row starts
    unsigned short* qb = (unsigned short*)(row + a.n + 1);     // [2][n] queue buffers
    const int tid = (int)threadIdx.x, lane = bq::lane_id();
    const unsigned wid = (unsigned)bq::bcast32(threadIdx.x >> 6);
    const unsigned shift = a.shift;
    const unsigned n = (unsigned)a.n;
    const unsigned long long t_start = bq::now_ticks();
    const unsigned none = (1u << (shift - 1u)) - 1u;

    for (unsigned v = tid; v < n; v += SMALL_WG)
        key[v] = v == (unsigned)a.src ? pack_key(0, none, shift) : KEY_INF;
    for (unsigned v = tid; v <= n; v += SMALL_WG) row[v] = (unsigned)a.off[v];
    if (tid < 3) {
        S.cnt[tid] = tid == 0 ? 1u : 0u;
        S.nhub[tid] = 0u;
    }
    if (tid == 0) {
        qb[0] = (unsigned short)a.src;
        S.neg = 0;
        S.err = bq::ERR_NONE;
        S.stop = 0u;
    }
    // weight range -> packing precondition and the negative-cycle bound
    long long lbound;
    {
        int lo, hi;
        weight_range((const int*)a.w, a.m, tid, SMALL_WG, lo, hi);
        for (int off = 32; off > 0; off >>= 1) {
            const int x = __shfl_xor(lo, off, 64), y = __shfl_xor(hi, off, 64);
            lo = x < lo ? x : lo;
            hi = y > hi ? y : hi;
        }
        if (lane == 0) {
            S.red[wid][0] = lo;
            S.red[wid][1] = hi;
        }
        __syncthreads();
        long long wmin = INT_MAX, wmax = INT_MIN, maxabs = 0;
        for (int i = 0; i < SMALL_WAVES; ++i) {
            wmin = S.red[i][0] < wmin ? S.red[i][0] : wmin;
            wmax = S.red[i][1] > wmax ? S.red[i][1] : wmax;
        }
        if (a.m > 0) {
            maxabs = wmax > -wmin ? wmax : -wmin;
            if (maxabs < 0) maxabs = -maxabs;
        }
        if ((double)a.n * (double)maxabs >= (double)(1ull << (62u - shift)))
            return SmallResult{0, bq::ERR_RANGE};
        lbound = (long long)(a.n - 1) * (wmin < 0 ? wmin : 0ll);
    }
    // lanes per item
    unsigned lg = 0;
    while (lg < 6u && ((long long)n << lg) < a.m) ++lg;
    const unsigned G = 1u << lg;
    const unsigned groups = SMALL_WG >> lg, group = (unsigned)tid >> lg, gl = (unsigned)tid & (G - 1u);
    const int hub_len = SMALL_HUB << lg;

    // below this key a candidate proves a negative cycle: its label is under
    // the certain lower bound (n - 1) * min w. A minus-infinity source counts
    // as -2^62, and since n * max |w| << shift is below 2^62 (checked above),
    // every candidate from it stays under that bound and none overflows
    const long long minus_inf = -(1ll << 62);
    const long long bkey = (long long)((unsigned long long)lbound << shift);
    const long long dmask = -1ll << shift;
    unsigned st_impr = 0, st_relax = 0;  // this lane's
    SweepWalk<false> walk{};
    int left = 64 * (int)n;  // items to the next walk that the others wait for

    for (unsigned it = 0;; ++it) {
        const unsigned cur = it % 3u, nxt = (it + 1u) % 3u, par = it & 1u;
        const unsigned NL = S.cnt[cur], NH = S.nhub[cur];
        // a stop raised in this sweep counts from the next one on, for every
        // wave alike
        if (NL + NH == 0u || S.stop - 1u < it) break;
        const unsigned short* q = qb + par * n;
        unsigned short* qn = qb + (par ^ 1u) * n;
        bool neg = false;
        // relax up to SMALL_U edges per lane and publish what improved
        // (base: the source's label and id, packed; a candidate is base + weight
        // at the label's place)
        auto relax = [&](auto uu, const int* tv, const long long* base, const int* w,
                         const bool* act, bool look) {
            constexpr int K = decltype(uu)::value;
            bool push[K];
            unsigned long long pm[K];
            unsigned np = 0;
#pragma unroll
            for (int r = 0; r < K; ++r) {
                push[r] = false;
                long long cand = base[r] + (long long)((unsigned long long)(long long)w[r] << shift);
                const bool below = act[r] && cand < bkey;
                neg |= below;
                if (below && a.neginf) cand = KEY_NEG;
                if (act[r] && (!look || cand < __hip_atomic_load(&key[tv[r]], __ATOMIC_RELAXED,
                                                                 __HIP_MEMORY_SCOPE_WORKGROUP))) {
                    const long long old = __hip_atomic_fetch_min(
                        &key[tv[r]], cand, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                    st_impr += cand < (old & dmask) ? 1u : 0u;
                    push[r] = cand < old && (old & 1ll) == 0;
                }
                pm[r] = bq::ballot(push[r]);
                np += (unsigned)__popcll(pm[r]);
            }
            if (np == 0u) return;
            unsigned at = 0;
            if (lane == 0) at = atomicAdd(&S.cnt[nxt], np);
            at = bq::bcast32(at);
#pragma unroll
            for (int r = 0; r < K; ++r) {
                if (push[r]) qn[at + (unsigned)bq::rank_in(pm[r])] = (unsigned short)tv[r];
                at += (unsigned)__popcll(pm[r]);
            }
            st.push += np;
        };
        // ---- long rows left by the sweep before: all waves together -------
        for (unsigned h = 0; h < NH; ++h) {
            const unsigned u = S.hub[par][h];
            const long long d = S.hub_d[par][h];
            const unsigned t = row[u + 1];
            for (unsigned e0 = row[u]; e0 < t; e0 += SMALL_WG * SMALL_U) {
                int tv[SMALL_U], w[SMALL_U];
                long long base[SMALL_U];
                bool act[SMALL_U];
#pragma unroll
                for (int r = 0; r < SMALL_U; ++r) {
                    const unsigned e = e0 + r * SMALL_WG + (unsigned)tid;
                    act[r] = e < t;
                    tv[r] = 0;
                    w[r] = 0;
                    base[r] = d;
                    if (act[r]) {
                        tv[r] = a.col[e];
                        w[r] = a.w[e];
                    }
                }
                relax(std::integral_constant<int, SMALL_U>{}, tv, base, w, act, true);
            }
        }
        // ---- the sweep's items ----------------------------------------------
        // K items per lane group from item b on
        auto take = [&](auto uu, unsigned b, bool look) {
            constexpr int K = decltype(uu)::value;
            unsigned u[K], s[K];
            long long base[K];
            int deg[K];
#pragma unroll
            for (int r = 0; r < K; ++r) {
                const unsigned i = b + (unsigned)r * groups + group;
                deg[r] = 0;
                u[r] = 0;
                s[r] = 0;
                base[r] = 0;
                if (i < NL) {
                    u[r] = q[i];
                    // clear q, then read the label: a wave's LDS operations
                    // are performed in order
                    if (gl == 0)
                        __hip_atomic_fetch_and(&key[u[r]], ~1ll, __ATOMIC_RELAXED,
                                               __HIP_MEMORY_SCOPE_WORKGROUP);
                }
            }
            __builtin_amdgcn_wave_barrier();
            int most = 0;
#pragma unroll
            for (int r = 0; r < K; ++r) {
                if (b + (unsigned)r * groups + group < NL) {
                    s[r] = row[u[r]];
                    deg[r] = (int)(row[u[r] + 1] - s[r]);
                    const long long k = __hip_atomic_load(&key[u[r]], __ATOMIC_RELAXED,
                                                          __HIP_MEMORY_SCOPE_WORKGROUP);
                    base[r] = (is_neg_key(k) ? minus_inf : k & dmask) |
                              (long long)((u[r] << 1) | 1u);
                }
                if (gl == 0) st_relax += (unsigned)deg[r];
                if (deg[r] > hub_len) {
                    unsigned at = SMALL_HUBS;
                    if (gl == 0) {
                        at = atomicAdd(&S.nhub[nxt], 1u);
                        if (at < SMALL_HUBS) {
                            S.hub[par ^ 1u][at] = u[r];
                            S.hub_d[par ^ 1u][at] = base[r];
                        } else {
                            atomicSub(&S.nhub[nxt], 1u);
                        }
                    }
                    at = (unsigned)__shfl((int)at, lane & ~(int)(G - 1u), 64);
                    if (at < SMALL_HUBS) deg[r] = 0;
                }
                most = deg[r] > most ? deg[r] : most;
            }
            for (int o = 0; __any(o < most); o += (int)G) {
                int tv[K], w[K];
                bool act[K];
#pragma unroll
                for (int r = 0; r < K; ++r) {
                    act[r] = o + (int)gl < deg[r];
                    tv[r] = 0;
                    w[r] = 0;
                    if (act[r]) {
                        const unsigned e = s[r] + (unsigned)o + gl;
                        tv[r] = a.col[e];
                        w[r] = a.w[e];
                    }
                }
                relax(uu, tv, base, w, act, look);
            }
        };
        // A sweep of at most one item per lane group takes them one at a time:
        // the instructions of empty places are half of its time. Waves past
        // the last item have nothing to do.
        const unsigned first = ((unsigned)tid & ~63u) >> lg;  // the wave's first group
        if (NL <= groups) {
            if (first < NL) take(std::integral_constant<int, 1>{}, 0u, false);
        } else {
            for (unsigned b = 0; b + first < NL; b += SMALL_U * groups)
                take(std::integral_constant<int, SMALL_U>{}, b, NL > 256u);
        }
        if (wid == 0) st.deq += NL;
        if (__any(neg)) {
            if (lane == 0) {
                S.neg = 1;
                if (!a.neginf) S.stop = it + 1u;
            }
        }
        // ---- negative-cycle search: one wave, a few steps per sweep. A cycle of
        // thousands of vertices changes before such a walk is round; so after
        // 64 n items (road meshes take 12 to 25 n) and every 16 n from there the
        // others wait at the barrier for one that goes as far as the parents lead.
        // Cycles of 2,000 in random graphs of 8,000 vertices took up to 680 ms, with
        // this 1 to 6.
        if (wid == SMALL_WAVES - 1u && it >= SWEEP_WALK_FROM) {
            const auto parent = [&](unsigned x) -> unsigned {
                const long long k = __hip_atomic_load(&key[x], __ATOMIC_RELAXED,
                                                      __HIP_MEMORY_SCOPE_WORKGROUP);
                return is_neg_key(k) ? none : (unsigned)(((unsigned long long)k >> 1) & none);
            };
            left -= (int)NL;
            int hit = -1;
            if (__builtin_expect(left < 0 && NL > 0u, 0)) {
                left = 16 * (int)n;
                walk.start(bq::bcast32((unsigned)q[it % NL]), parent);
                ++st.walk;
                hit = walk.advance(a, parent, 3u * n);
            }
            if (!walk.on && NL > 0u) {
                walk.start(bq::bcast32((unsigned)q[it % NL]), parent);
                ++st.walk;
            }
            if (hit < 0) hit = walk.advance(a, parent, SWEEP_WALK_STEPS);
            if (hit >= 0) {
                if (lane == 0) {
                    S.neg = 1;
                    if (!a.neginf) S.stop = it + 1u;
                    else {
                        const long long old = __hip_atomic_fetch_min(
                            &key[hit], KEY_NEG, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                        if (KEY_NEG < old && (old & 1ll) == 0)
                            qn[atomicAdd(&S.cnt[nxt], 1u)] = (unsigned short)hit;
                    }
                }
            }
        }
        if (tid == 0) {
            // the words of the sweep after next were last read before the
            // latest barrier
            S.cnt[(it + 2u) % 3u] = 0u;
            S.nhub[(it + 2u) % 3u] = 0u;
            if (bq::now_ticks() - t_start > a.deadline) {
                S.err = bq::ERR_TIMEOUT;
                S.stop = it + 1u;
            }
        }
        __syncthreads();
    }
    for (int off = 32; off > 0; off >>= 1) st_relax += (unsigned)__shfl_xor((int)st_relax, off, 64);
    st.impr += st_impr;
    st.relax += st_relax;
    // ---- unpack ----------------------------------------------------------
    const long long dmax = KEY_INF >> shift;
    unsigned long long redges = 0;
    for (unsigned v = tid; v < n; v += SMALL_WG) {
        const long long k = key[v], d = k >> shift;
        const bool minus = is_neg_key(k), seen = minus || d != dmax;
        dist[v] = minus ? LLONG_MIN : (seen ? d : LLONG_MAX);
        if (pred)
            pred[v] = (seen && !minus && v != (unsigned)a.src)
                          ? (int)(((unsigned long long)k >> 1) & none)
                          : -1;
        if (reached && seen) redges += (unsigned long long)(row[v + 1] - row[v]);
    }
    if (reached) {
        for (int off = 32; off > 0; off >>= 1) redges += __shfl_xor(redges, off, 64);
        if (lane == 0 && redges) bq::add_rlx(reached, redges);
    }
    return SmallResult{S.neg, S.err};
}

}  // namespace
