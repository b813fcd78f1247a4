// The sweep form of the queue-driven Bellman-Ford (Section III.C): the same
// keys, relaxations and results as the asynchronous solver in
// sssp_device.hpp, with the queue drained in sweeps.
//
// The queue is two buffers of items. A sweep takes every item one buffer
// holds, and the vertices it improves are published to the other; the
// workgroups of a query (its gang) meet at a barrier between sweeps, and an
// empty buffer ends the solve. So no operation waits for a slot and no head,
// count or pending word exists: the items of a sweep are shared out by
// position (the dequeue costs no atomic), and a publish is one atomic add on a
// segment's tail word for up to 64 vertices.
//
// Why sweeps: the asynchronous form pays about six dependent memory-side
// round trips per batch (three broker reservations, slot reads, staging and
// publish; 9 us per tree edge on a mesh), and its waves must be few, since
// more of them scan labels before they settle. A sweep costs one
// barrier (1.5-2 us for 256 workgroups), about 6 us in all when it holds few
// items, and runs every wave of the chip. Counted on the CPU: RMAT-20 needs 15
// sweeps and 2.4-3.3 relaxations per reached edge, a random graph of 200k
// vertices 25 sweeps and 3.4-3.9.
//
// Items. A light item is a vertex whose row has at most C = 2^chunk_log
// edges. A longer row is published as ceil(degree / C) chunk items
// (vertex, chunk), so that every wave of the next sweep shares it. The key's
// q bit keeps a vertex from being published twice: whoever lowers a key whose
// q was 0 publishes the vertex, and reading an item clears q and returns the
// label in one atomic, so a label that fell earlier in the same sweep is used
// at once. Each chunk item of a row clears q when it reads the label, so no
// drop after any chunk's read can go unpublished; a drop between two chunks'
// reads may then find q = 0 while the row is already in the next buffer, and
// `stamp` (the sweep the row was last published for) drops that second
// publish. So a buffer holds each vertex at most once, and the buffers' sizes
// follow from n and m alone.
//
// Copying the labels to an array of their own between sweeps, for the looks
// before the atomics to read, took the coherence traffic out of the looks
// (104 against 32 G random relaxations/s on 200k keys in isolation), but with
// labels one sweep old the work ratio rose (random graph of 1M vertices 3.6 ->
// 4.2, RMAT-20 3.0 -> 3.4) and the solves took 1.28 against 1.15 ms and 0.98
// against 0.92 ms: the sweeps are bound by the rows' and keys' lines.
//
// Memory ordering: the words shared inside a launch (keys, tails, items,
// stamps, barrier words) are read and written by agent-scope atomics, which are
// performed at the device's coherence point; a wave waits for its own
// (s_waitcnt) before its workgroup arrives at the barrier. The CSR is
// read-only and takes ordinary cached loads.
#pragma once
#include <hip/hip_runtime.h>
#include <limits.h>

#include "sssp_device.hpp"
#include "sssp_init.hpp"
#include "sssp_strip.hpp"

namespace {

constexpr int SWEEP_WG = 1024;
constexpr int SWEEP_WAVES = SWEEP_WG / 64;
constexpr int SWEEP_U = 4;         // edges per lane per scan step
constexpr int SWEEP_OUT = 512;     // LDS push buffer per wave
constexpr int SWEEP_TILE = 2048;   // edges of a batch mapped to their items at a time
constexpr unsigned SWEEP_LIGHT = 16;  // light and chunk items of a batch at most:
constexpr unsigned SWEEP_CHUNKS = 4;  // see sweep_instance
constexpr unsigned long long SWEEP_STOP = ~0ull;  // barrier epoch: leave

// Barrier and tail words of one query, each on its own line.
struct SweepCtl {
    bq::Word tail[3][MAX_SEG];  // chunk items << 32 | light items of a buffer's segment
    bq::Word arrive[8];         // arrivals of the gang's members, by rank mod 8 (32 bits)
    bq::Word root;              // full groups (32 bits)
    bq::Word joined;            // workgroups that have asked to take part
    bq::Word go;                // last sweep released << 32 | its members
};

struct SweepArgs {
    BQ_GLOBAL SweepCtl* ctl;
    BQ_GLOBAL unsigned* light;             // [2][nseg][cap_light]
    BQ_GLOBAL unsigned long long* chunk;   // [2][nseg][cap_chunk]
    BQ_GLOBAL unsigned* stamp;             // [n] used for chunked rows only
    BQ_GLOBAL unsigned* longp;             // per init block: its longest row (note_row)
    unsigned cap_light;
    unsigned cap_chunk;
    StripArgs p;  // of the strip form, which is tried first; p.ctl null: it is not
};

struct SweepWave {
    long long du[64];
    long long eb[64];      // row start minus the item's first position in the batch
    unsigned pu[64];       // vertex (parent field of candidates)
    int fan[64];
    unsigned hv[64];
    unsigned out[SWEEP_OUT];
    alignas(4) unsigned char own[SWEEP_TILE];
    WalkSum walk;
};

template <int WAVES>
struct SweepLds {
    SweepWave w[WAVES];
    long long red[WAVES][3];
    unsigned long long stats[bq::ST_N];
    unsigned nout[WAVES];  // pushes each wave holds at the end of a sweep
    unsigned long long base;
    unsigned long long go;
    unsigned rank;
    int walk_hit;        // gang_walk: a vertex of a negative cycle, or -1
    unsigned walk_over;  // gang_walk: the solve is over
};

__device__ __forceinline__ void sweep_stop(const SweepArgs& f) {
    __hip_atomic_fetch_max(&f.ctl->go.v, SWEEP_STOP, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// A gang's members. A workgroup joins a solve when it gets to run and takes
// part from the next sweep on; nobody waits for one that has not started, so
// launches that share the chip (other streams, other gangs) cannot hold each
// other up. The first to join gives the others 10 us before the first sweep.
struct SweepGang {
    unsigned rank, members, sweep;
};

// Join the solve (up to `want` workgroups). False when it is over, or stopped.
// Every wait ends at the solve's deadline at the latest.
template <int WAVES>
__device__ bool gang_join(const SolveArgs& a, const SweepArgs& f, unsigned want, SweepGang& g,
                          SweepLds<WAVES>& S, unsigned long long t_start) {
    if (threadIdx.x == 0) {
        BQ_GLOBAL SweepCtl* c = f.ctl;
        const unsigned rank = (unsigned)bq::add_rlx(&c->joined.v, 1ull);
        unsigned long long go = SWEEP_STOP;
        const unsigned long long t0 = bq::now_ticks();
        if (rank == 0) {
            unsigned long long j;
            do j = bq::ld_rlx(&c->joined.v);
            while (j < want && bq::now_ticks() - t0 < 1000ull);
            const unsigned long long was = __hip_atomic_fetch_max(
                &c->go.v, j, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            go = was == SWEEP_STOP ? was : j;
        } else {
            for (unsigned it = 1;; ++it) {
                go = bq::ld_rlx(&c->go.v);
                if (go == SWEEP_STOP || (unsigned)go > rank) break;
                if ((it & 63u) == 0u && bq::now_ticks() - t_start > a.deadline) {
                    go = SWEEP_STOP;
                    break;
                }
            }
        }
        S.rank = rank;
        S.go = go;
    }
    __syncthreads();
    g.rank = S.rank;
    g.members = (unsigned)S.go;
    g.sweep = (unsigned)(S.go >> 32);
    const bool in = S.go != SWEEP_STOP;
    __syncthreads();
    return in;
}

// A member's arrival after its sweep and its wait for the next one, by one
// thread: the next value of `go`.
__device__ unsigned long long gang_meet(const SolveArgs& a, const SweepArgs& f, const SweepGang& g,
                                        unsigned long long t_start) {
    BQ_GLOBAL SweepCtl* c = f.ctl;
    const unsigned grp = g.rank & 7u;
    const unsigned ng = g.members < 8u ? g.members : 8u, gs = (g.members + 7u - grp) >> 3;
    const unsigned next = g.sweep + 1u;
    if (atomicInc((unsigned*)&c->arrive[grp].v, gs - 1u) == gs - 1u) {
        const unsigned long long j = bq::ld_rlx(&c->joined.v);
        if (atomicInc((unsigned*)&c->root.v, ng - 1u) == ng - 1u) {
            const unsigned m = (unsigned)j > g.members ? (unsigned)j : g.members;
            __hip_atomic_fetch_max(&c->go.v, ((unsigned long long)next << 32) | m,
                                   __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
    const unsigned long long t0 = bq::now_ticks();
    unsigned long long go;
    for (unsigned it = 1;; ++it) {
        go = bq::ld_rlx(&c->go.v);
        if ((unsigned)(go >> 32) >= next) break;
        if ((it & 63u) == 0u) {
            const unsigned long long t = bq::now_ticks();
            if (t - t0 > a.limit || t - t_start > a.deadline) {
                bq::raise_error(a.q, bq::ERR_TIMEOUT);
                sweep_stop(f);
            }
        }
    }
    if (go != SWEEP_STOP && bq::now_ticks() - t_start > a.deadline) {
        bq::raise_error(a.q, bq::ERR_TIMEOUT);
        sweep_stop(f);
        go = SWEEP_STOP;
    }
    return go;
}

// The members meet after a sweep; returns false when the solve was stopped,
// else g is the next sweep with the members it has. Arrivals go to one
// self-resetting word per rank mod 8, the last of a group arrives at the root,
// the last of the groups releases `go`, which is the only word the waiting
// workgroups read (polling a word slows the atomics on it). 256 workgroups on
// one word took 4.2 us; 64 took 1.5 us. Every wait ends: past the wait limit
// or the solve's deadline the waiter raises the timeout and releases everyone
// with SWEEP_STOP.
template <int WAVES>
__device__ bool gang_barrier(const SolveArgs& a, const SweepArgs& f, SweepGang& g,
                             SweepLds<WAVES>& S, unsigned long long t_start) {
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    __syncthreads();
    if (threadIdx.x == 0) S.go = gang_meet(a, f, g, t_start);
    __syncthreads();
    g.members = (unsigned)S.go;
    ++g.sweep;
    return S.go != SWEEP_STOP;
}

// Publish the wave's improved vertices L.out[0, cnt) for sweep `next`, one
// atomic per 64: light items, and the chunk items of longer rows.
__device__ __forceinline__ void sweep_publish(const SolveArgs& a, const SweepArgs& f, SweepWave& L,
                                              int cnt, unsigned next, unsigned home,
                                              bool long_rows, WaveStats& st) {
    const int lane = bq::lane_id();
    BQ_GLOBAL unsigned long long* tail = &f.ctl->tail[next % 3u][home].v;
    const unsigned long long part = (unsigned long long)((next & 1u) * a.nseg + home);
    BQ_GLOBAL unsigned* light = f.light + part * f.cap_light;
    BQ_GLOBAL unsigned long long* chunk = f.chunk + part * f.cap_chunk;
    __builtin_amdgcn_wave_barrier();
    for (int c0 = 0; c0 < cnt; c0 += 64) {
        const int i = c0 + lane;
        bool live = i < cnt;
        const unsigned v = live ? L.out[i] : 0u;
        int nch = 0;
        if (long_rows) {
            if (live) {
                const long long deg = a.off[v + 1] - a.off[v];
                if (deg > (1ll << a.chunk_log))
                    nch = (int)((deg + (1ll << a.chunk_log) - 1) >> a.chunk_log);
            }
            if (nch > 0) {
                const unsigned was = __hip_atomic_fetch_max(&f.stamp[v], next, __ATOMIC_RELAXED,
                                                            __HIP_MEMORY_SCOPE_AGENT);
                if (was == next) {  // already in the next buffer
                    nch = 0;
                    live = false;
                }
            }
        }
        const unsigned long long lm = bq::ballot(live && nch == 0);
        const int nl = __popcll(lm);
        int incl = 0, ntc = 0;
        if (long_rows && __any(nch > 0)) {
            incl = bq::wave_incl_scan(nch);
            ntc = bq::lane63(incl);
        }
        unsigned long long base = 0;
        if (lane == 0 && (nl | ntc) != 0)
            base = bq::add_rlx(tail, ((unsigned long long)ntc << 32) | (unsigned long long)nl);
        base = bq::bcast64(base);
        if (live && nch == 0)
            bq::st_rlx(&light[(unsigned)base + (unsigned)bq::rank_in(lm)], v);
        if (ntc > 0) {
            const unsigned cb = (unsigned)(base >> 32);
            L.fan[lane] = incl - nch;
            L.hv[lane] = v;
            __builtin_amdgcn_wave_barrier();
            for (int k = lane; k < ntc; k += 64) {
                int lo = 0, hi = 64;  // largest index with fan <= k: the row of chunk k
                while (hi - lo > 1) {
                    const int mid = (lo + hi) >> 1;
                    if (L.fan[mid] <= k) lo = mid;
                    else hi = mid;
                }
                bq::st_rlx(&chunk[cb + (unsigned)k],
                           ((unsigned long long)(k - L.fan[lo]) << 32) | L.hv[lo]);
            }
            __builtin_amdgcn_wave_barrier();
            st.fan += (unsigned long long)ntc;
        }
        st.push += (unsigned long long)__popcll(bq::ballot(live));
    }
    __builtin_amdgcn_wave_barrier();
}

// The same for all waves of the workgroup with one atomic (graphs without
// chunked rows): in a wide sweep 3,000 waves that each add to one of 8 tail
// words wait up to 5 us for them.
template <int WAVES>
__device__ void sweep_publish_wg(const SolveArgs& a, const SweepArgs& f, SweepLds<WAVES>& S,
                                 unsigned wid, int cnt, unsigned next, unsigned home,
                                 WaveStats& st) {
    const int lane = bq::lane_id();
    if (lane == 0) S.nout[wid] = (unsigned)cnt;
    __syncthreads();
    unsigned before = 0, total = 0;
    for (unsigned i = 0; i < (unsigned)WAVES; ++i) {
        const unsigned x = S.nout[i];
        before += i < wid ? x : 0u;
        total += x;
    }
    if (total == 0u) return;  // workgroup-uniform
    if (threadIdx.x == 0)
        S.base = bq::add_rlx(&f.ctl->tail[next % 3u][home].v, (unsigned long long)total);
    __syncthreads();
    const unsigned base = (unsigned)S.base + before;
    BQ_GLOBAL unsigned* light =
        f.light + (unsigned long long)((next & 1u) * a.nseg + home) * f.cap_light;
    for (int i = lane; i < cnt; i += 64) bq::st_rlx(&light[base + (unsigned)i], S.w[wid].out[i]);
    st.push += (unsigned long long)cnt;
}

// Map edges [T0, T0 + tl) of the batch to their items: every item with edges
// marks its first one, then a running maximum carries the marks on, 4 bytes
// per lane and one wave scan per 256 edges. `cnt` and `pre` are the lane's
// item (its edges and its first position in the batch).
__device__ __forceinline__ void sweep_map(SweepWave& L, int T0, int tl, int cnt, int pre) {
    const int lane = bq::lane_id();
    unsigned* own32 = reinterpret_cast<unsigned*>(L.own);
    const int words = (tl + 3) >> 2;
    for (int i = lane; i < words; i += 64) own32[i] = 0u;
    __builtin_amdgcn_wave_barrier();
    const int rel = pre - T0;
    if (cnt > 0 && rel > 0 && rel < tl) L.own[rel] = (unsigned char)lane;
    // the item that holds edge T0
    unsigned carry = 63u - (unsigned)__clzll(bq::ballot(cnt > 0 && rel <= 0));
    __builtin_amdgcn_wave_barrier();
    for (int w0 = 0; w0 < words; w0 += 64) {
        const int wi = w0 + lane;
        const unsigned v = wi < words ? own32[wi] : 0u;
        unsigned b0 = v & 255u, b1 = (v >> 8) & 255u, b2 = (v >> 16) & 255u, b3 = v >> 24;
        b1 = b1 > b0 ? b1 : b0;
        b2 = b2 > b1 ? b2 : b1;
        b3 = b3 > b2 ? b3 : b2;
        const unsigned incl = bq::wave_incl_max(b3);
        unsigned prev = bq::wave_shr1(incl);  // lane 0 reads 0
        prev = prev > carry ? prev : carry;
        b0 = b0 > prev ? b0 : prev;
        b1 = b1 > prev ? b1 : prev;
        b2 = b2 > prev ? b2 : prev;
        b3 = b3 > prev ? b3 : prev;
        if (wi < words) own32[wi] = b0 | (b1 << 8) | (b2 << 16) | (b3 << 24);
        const unsigned last = (unsigned)bq::lane63((int)incl);
        carry = last > carry ? last : carry;
    }
    __builtin_amdgcn_wave_barrier();
}

// Segment and index in it of item g of a sweep; lane s of `pre` holds the
// number of items in the segments before s. Empty segments share their
// prefix with the next one, which wins.
struct SweepSlot {
    unsigned seg, i;
};
__device__ __forceinline__ SweepSlot sweep_slot(unsigned nseg, unsigned pre, unsigned g) {
    unsigned seg = 0, first = 0;
    for (unsigned s = 1; s < nseg; ++s) {
        const unsigned p = (unsigned)__builtin_amdgcn_readlane((int)pre, (int)s);
        if (p <= g) {
            seg = s;
            first = p;
        }
    }
    return SweepSlot{seg, g - first};
}

// Whether the member of rank 1 walks for good (gang_walk). A solve that has so
// many sweeps has a long chain of steps, where a member less costs little, or a
// negative cycle. (RMAT and random graphs take 15 to 30 sweeps.)
__device__ __forceinline__ bool gang_walks(const SweepGang& g) {
    const unsigned from = g.members >= 64u ? 64u : (g.members >= 8u ? 512u : 4096u);
    return g.members >= 2u && g.sweep >= from;
}

// The member that searches for negative cycles while the others sweep. Its first
// wave meets them at every sweep, at once, with nothing done; the others walk
// from vertices drawn at random and wait for nobody. A few moves a sweep are
// enough to close a short cycle, but a sweep of a wide queue takes as long as a
// hundred moves, and on long cycles the parents changed before such a walk was
// round: random graphs of 15k to 400k vertices with a cycle of 2,000 to 8,000
// vertices took 3 to 850 ms, with it 1 to 7. (A random graph of 200k vertices takes
// 439 us for 432: its 29 sweeps end before this, but the loop has more to hold.
// Called instead of inlined it took 546.)
template <int WAVES>
__device__ __forceinline__ void gang_walk(const SolveArgs& a, const SweepArgs& f, SweepGang& g,
                                          SweepLds<WAVES>& S, unsigned wid, unsigned home,
                                          bool long_rows, WaveStats& st,
                                          unsigned long long t_start) {
    const int lane = bq::lane_id();
    SweepWave& L = S.w[wid];
    if (threadIdx.x == 0) {
        S.walk_hit = -1;
        S.walk_over = 0u;
    }
    __syncthreads();
    if (wid == 0u) {
        bool flagged = false;
        for (;;) {
            int hit = -1;
            if (lane == 0) hit = atomicExch(&S.walk_hit, -1);
            hit = (int)bq::bcast32((unsigned)hit);
            if (hit >= 0) {
                if (lane == 0 && !flagged) bq::st_rlx(&a.q.ctrl->negcycle.v, 1ull);
                flagged = true;
                if (!a.neginf) {
                    if (lane == 0) {
                        bq::st_rlx(&a.q.ctrl->abort.v, 1ull);
                        sweep_stop(f);
                    }
                } else {
                    // a mark is published before this member meets the others
                    long long old = 0;
                    if (lane == 0)
                        old = __hip_atomic_fetch_min(&a.key[hit], KEY_NEG, __ATOMIC_RELAXED,
                                                     __HIP_MEMORY_SCOPE_AGENT);
                    old = (long long)bq::bcast64((unsigned long long)old);
                    if (KEY_NEG < old && (old & 1ll) == 0) {
                        if (lane == 0) L.out[0] = (unsigned)hit;
                        sweep_publish(a, f, L, 1, g.sweep + 1u, home, long_rows, st);
                    }
                }
            }
            asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
            unsigned long long go = 0;
            if (lane == 0) go = gang_meet(a, f, g, t_start);
            go = bq::bcast64(go);
            if (go == SWEEP_STOP) break;
            g.members = (unsigned)go;
            ++g.sweep;
        }
        if (lane == 0)
            __hip_atomic_store(&S.walk_over, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    } else {
        const auto parent = [&](unsigned x) { return parent_of(a, (int)x); };
        SweepWalk<true> walk{};
        unsigned draw = wid * 0x9E3779B9u + g.sweep;
        while (__hip_atomic_load(&S.walk_over, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) ==
               0u) {
            if (!walk.on) {
                draw = draw * 1664525u + 1013904223u;
                walk.start((unsigned)(((unsigned long long)draw * (unsigned)a.n) >> 32), parent);
                ++st.walk;
            }
            const int hit = walk.advance(a, parent, 32u, &L.walk);
            if (hit >= 0 && lane == 0) atomicExch(&S.walk_hit, hit);
        }
    }
    __syncthreads();
}

// One gang's solve of one query; up to `want` workgroups call it with the same
// arguments. Returns 1 when the queue ran empty, -1 when the solve was stopped
// (error or negative cycle) or over before this workgroup joined.
template <int WAVES>
__device__ __forceinline__ int sweep_instance(const SolveArgs& a, const SweepArgs& f,
                                              unsigned want, SweepLds<WAVES>& S, WaveStats& st) {
    const int lane = bq::lane_id();
    const unsigned wid = (unsigned)bq::bcast32(threadIdx.x >> 6);
    SweepWave& L = S.w[wid];
    const unsigned shift = a.shift;
    const long long C = 1ll << a.chunk_log;
    const unsigned long long t_start = bq::ld_rlx(&a.q.ctrl->aux[4].v);

    // weight range -> packing precondition and the negative-cycle bound; and
    // whether any row is chunked
    bool long_rows;
    long long lbound;
    {
        const int parts = (int)bq::ld_rlx(&a.q.ctrl->aux[0].v);
        int lo = INT_MAX, hi = INT_MIN;
        unsigned lr = 0;
        for (int i = (int)threadIdx.x; i < parts; i += WAVES * 64) {
            const int x = a.wrange[2 * i], y = a.wrange[2 * i + 1];
            lo = x < lo ? x : lo;
            hi = y > hi ? y : hi;
            lr |= f.longp[i] > (unsigned long long)C ? 1u : 0u;
        }
        for (int off = 32; off > 0; off >>= 1) {
            const int x = __shfl_xor(lo, off, 64), y = __shfl_xor(hi, off, 64);
            lo = x < lo ? x : lo;
            hi = y > hi ? y : hi;
        }
        const bool any_long = __any(lr != 0u);
        if (lane == 0) {
            S.red[wid][0] = lo;
            S.red[wid][1] = hi;
            S.red[wid][2] = any_long ? 1 : 0;
        }
        __syncthreads();
        long long wmin = INT_MAX, wmax = INT_MIN, lg = 0;
        for (int i = 0; i < WAVES; ++i) {
            wmin = S.red[i][0] < wmin ? S.red[i][0] : wmin;
            wmax = S.red[i][1] > wmax ? S.red[i][1] : wmax;
            lg |= S.red[i][2];
        }
        long_rows = lg != 0;
        long long maxabs = 0;
        if (a.m > 0) {
            maxabs = wmax > -wmin ? wmax : -wmin;
            if (maxabs < 0) maxabs = -maxabs;
        }
        // every label of a simple path satisfies |d| <= (n-1) * max|w|; a
        // candidate is at most one more edge away from a checked label
        if ((double)a.n * (double)maxabs >= (double)(1ull << (62u - shift))) {
            if (threadIdx.x == 0) bq::raise_error(a.q, bq::ERR_RANGE);
            return -1;  // every workgroup of the gang sees the same range
        }
        lbound = (long long)(a.n - 1) * (wmin < 0 ? wmin : 0ll);
    }

    SweepGang g;
    if (!gang_join<WAVES>(a, f, want, g, S, t_start)) return -1;
    const unsigned home = g.rank % a.nseg;
    SweepWalk<true> walk{};
    bool flagged = false;  // marking mode: this wave already raised negcycle
    long long to_long = 16ll * a.n;  // items to the next long walk
    int result = -1;

    while (true) {
        const unsigned it = g.sweep;
        const bool walks = gang_walks(g);
        const unsigned workers = g.members - (walks ? 1u : 0u), W = workers * WAVES;
        // consecutive batches go to different workgroups, so a short sweep
        // spreads over the gang's CUs
        const unsigned gw = wid * workers + g.rank - (walks && g.rank > 1u ? 1u : 0u);
        // ---- the sweep's items, by segment ------------------------------
        unsigned long long tw = 0;
        if ((unsigned)lane < a.nseg) tw = bq::ld_rlx(&f.ctl->tail[it % 3u][lane].v);
        const int incl_l = bq::wave_incl_scan((int)(unsigned)tw);
        const unsigned NL = (unsigned)bq::lane63(incl_l);
        const unsigned pre_l = (unsigned)incl_l - (unsigned)tw;
        unsigned NC = 0, pre_c = 0;
        if (long_rows) {
            const int incl_c = bq::wave_incl_scan((int)(tw >> 32));
            NC = (unsigned)bq::lane63(incl_c);
            pre_c = (unsigned)incl_c - (unsigned)(tw >> 32);
        }
        if (NL + NC == 0u) {
            if (g.rank == 0 && threadIdx.x == 0) sweep_stop(f);  // nobody joins any more
            result = 1;
            break;
        }
        if (walks && g.rank == 1u) {
            gang_walk<WAVES>(a, f, g, S, wid, home, long_rows, st, t_start);
            break;
        }
        // the buffer after next is empty; its words were last read before the
        // latest barrier
        if (g.rank == 0 && threadIdx.x < a.nseg)
            bq::st_rlx(&f.ctl->tail[(it + 2u) % 3u][threadIdx.x].v, 0ull);
        const unsigned long long part0 = (unsigned long long)((it & 1u) * a.nseg);
        // batches: chunk items first (the hubs' rows: most labels fall through
        // them), then light items; sized so that every wave has one, and small
        // enough that the labels, which are read when a batch begins, are fresh
        // when its last row is scanned: with up to 64 light and 32 chunk items
        // RMAT-20 relaxed 2.97 times its edges and took 916 us, with 16 and 4
        // 2.27 times and 796 us (a random graph of 1M vertices 3.67 and 1,110
        // against 3.32 and 1,049); 8 and 4 scan no faster (2.21, 806 us).
        unsigned cbs = (NC + W - 1u) / W;
        cbs = cbs > SWEEP_CHUNKS ? SWEEP_CHUNKS : cbs;
        unsigned lbs = (NL + W - 1u) / W;
        lbs = lbs > SWEEP_LIGHT ? SWEEP_LIGHT : lbs;
        const unsigned nbc = cbs ? (NC + cbs - 1u) / cbs : 0u;
        const unsigned nbl = lbs ? (NL + lbs - 1u) / lbs : 0u;
        // a sweep of few items relaxes without the look at the key before the
        // atomic: there the look is one more round trip, not saved traffic
        const bool wide = NL + 32u * NC > 2u * W;
        int nout = 0;
        bool ok = true;
        for (unsigned b = gw; b < nbc + nbl && ok; b += W) {
            const bool chunks = b < nbc;
            const unsigned b0 = chunks ? b * cbs : (b - nbc) * lbs;
            const unsigned lim = chunks ? NC : NL, bs = chunks ? cbs : lbs;
            const unsigned e = lim - b0 < bs ? lim - b0 : bs;
            // ---- stage: lane i holds item b0 + i -------------------------
            int cnt = 0;
            long long eb = 0;
            const SweepSlot at = sweep_slot(a.nseg, chunks ? pre_c : pre_l, b0 + (unsigned)lane);
            if ((unsigned)lane < e) {
                unsigned v;
                long long j = -1;
                if (chunks) {
                    const unsigned long long x =
                        bq::ld_rlx(&f.chunk[(part0 + at.seg) * f.cap_chunk + at.i]);
                    v = (unsigned)x;
                    j = (long long)(x >> 32);
                } else {
                    v = bq::ld_rlx(&f.light[(part0 + at.seg) * f.cap_light + at.i]);
                }
                const long long old = __hip_atomic_fetch_and(
                    &a.key[v], ~1ll, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                long long t = a.off[v + 1];
                eb = a.off[v];
                if (j >= 0) {
                    eb += j << a.chunk_log;
                    t = t < eb + C ? t : eb + C;
                }
                cnt = (int)(t - eb);
                L.du[lane] = old >> shift;
                L.pu[lane] = v;
            }
            const int incl = bq::wave_incl_scan(cnt);
            const int pre = incl - cnt;
            const int total = bq::lane63(incl);
            if ((unsigned)lane < e) L.eb[lane] = eb - pre;
            ++st.batch;
            st.deq += e;
            st.relax += (unsigned long long)total;
            // ---- scan the concatenated rows ------------------------------
            for (int T0 = 0; T0 < total && ok; T0 += SWEEP_TILE) {
                const int tl = total - T0 < SWEEP_TILE ? total - T0 : SWEEP_TILE;
                sweep_map(L, T0, tl, cnt, pre);
                for (int t0 = 0; t0 < tl; t0 += 64 * SWEEP_U) {
                    int tv[SWEEP_U], w[SWEEP_U], idx[SWEEP_U];
                    long long cand[SWEEP_U], cd[SWEEP_U], seen[SWEEP_U], old[SWEEP_U];
                    bool live[SWEEP_U];
#pragma unroll
                    for (int r = 0; r < SWEEP_U; ++r) {
                        const int t = t0 + r * 64 + lane;
                        live[r] = t < tl;
                        tv[r] = 0;
                        w[r] = 0;
                        idx[r] = 0;
                        if (live[r]) {
                            idx[r] = (int)L.own[t];
                            const long long edge = L.eb[idx[r]] + (T0 + t);
                            tv[r] = a.col[edge];
                            w[r] = a.w[edge];
                        }
                    }
#pragma unroll
                    for (int r = 0; r < SWEEP_U; ++r)
                        seen[r] = live[r] && wide ? bq::ld_rlx(&a.key[tv[r]]) : LLONG_MAX;
#pragma unroll
                    for (int r = 0; r < SWEEP_U; ++r) {
                        cd[r] = L.du[idx[r]] + (long long)w[r];
                        cand[r] = pack_key(cd[r], L.pu[idx[r]], shift);
                        // marking mode: a candidate below the certain lower
                        // bound (or from a minus-infinity source) proves that a
                        // negative cycle reaches the target
                        if (a.neginf && cd[r] < lbound) cand[r] = KEY_NEG;
                        live[r] = live[r] && cand[r] < seen[r];
                        old[r] = live[r] ? __hip_atomic_fetch_min(&a.key[tv[r]], cand[r],
                                                                  __ATOMIC_RELAXED,
                                                                  __HIP_MEMORY_SCOPE_AGENT)
                                         : LLONG_MIN;
                    }
                    bool neg = false;
#pragma unroll
                    for (int r = 0; r < SWEEP_U; ++r) {
                        const bool won = live[r] && cand[r] < old[r];
                        const bool dropped = won && cd[r] < (old[r] >> shift);
                        st.impr += dropped;
                        neg |= dropped && cd[r] < lbound;
                        const bool push = won && (old[r] & 1ll) == 0;
                        const unsigned long long pm = bq::ballot(push);
                        if (push) L.out[nout + bq::rank_in(pm)] = (unsigned)tv[r];
                        nout += __popcll(pm);
                    }
                    if (__any(neg)) {
                        if (lane == 0 && !flagged) bq::st_rlx(&a.q.ctrl->negcycle.v, 1ull);
                        flagged = true;
                        if (!a.neginf) {
                            if (lane == 0) {
                                bq::st_rlx(&a.q.ctrl->abort.v, 1ull);
                                sweep_stop(f);
                            }
                            ok = false;
                            break;
                        }
                    }
                    if (nout > SWEEP_OUT - 64 * SWEEP_U) {
                        sweep_publish(a, f, L, nout, it + 1u, home, long_rows, st);
                        nout = 0;
                    }
                }
            }
        }
        // ---- negative-cycle search ---------------------------------------
        if (gw + SWEEP_WALKERS >= W && it >= SWEEP_WALK_FROM && ok) {
            const auto parent = [&](unsigned x) { return parent_of(a, (int)x); };
            // a few moves a sweep; in a small gang, whose sweeps are long, after
            // 16 n items one walk at up to 2,048 moves a sweep (1.5 ms) until it ends,
            // while the others wait: 64 random graphs of 15k vertices with a cycle of
            // 2,000 took 150 ms, with this 5.4, 256 of them 550 and 20; 64 permuted
            // meshes of 300 x 300 (22 n items each) 28.1 and 28.4
            int rounds = 1;
            if (g.members < 64u) {
                const bool first = to_long >= 0;
                to_long -= (long long)NL + NC;
                if (to_long < 0) {
                    rounds = SWEEP_WALK_LONG;
                    walk.on = walk.on && !first;
                }
            }
            if (!walk.on) {
                const unsigned k = (it + gw) % (NL > 0 ? NL : NC);
                const SweepSlot at = sweep_slot(a.nseg, NL > 0 ? pre_l : pre_c, k);
                walk.start(bq::bcast32(
                    NL > 0 ? bq::ld_rlx(&f.light[(part0 + at.seg) * f.cap_light + at.i])
                           : (unsigned)bq::ld_rlx(&f.chunk[(part0 + at.seg) * f.cap_chunk + at.i])),
                    parent);
                ++st.walk;
            }
            int hit;
            do {
                hit = walk.advance(a, parent, SWEEP_WALK_STEPS, &L.walk);
                rounds -= walk.left != 0u ? (int)SWEEP_WALK_SUMS / (int)SWEEP_WALK_STEPS : 1;
            } while (walk.on && rounds > 0);
            if (to_long < 0 && !walk.on) to_long = 16ll * a.n;
            if (hit >= 0) {
                if (lane == 0 && !flagged) bq::st_rlx(&a.q.ctrl->negcycle.v, 1ull);
                flagged = true;
                if (!a.neginf) {
                    if (lane == 0) {
                        bq::st_rlx(&a.q.ctrl->abort.v, 1ull);
                        sweep_stop(f);
                    }
                } else {
                    // the cycle's vertex becomes minus infinity and spreads it
                    // through the queue like any lowered label
                    if (nout > 0) sweep_publish(a, f, L, nout, it + 1u, home, long_rows, st);
                    long long old = 0;
                    if (lane == 0)
                        old = __hip_atomic_fetch_min(&a.key[hit], KEY_NEG, __ATOMIC_RELAXED,
                                                     __HIP_MEMORY_SCOPE_AGENT);
                    old = (long long)bq::bcast64((unsigned long long)old);
                    nout = (KEY_NEG < old && (old & 1ll) == 0) ? 1 : 0;
                    if (lane == 0) L.out[0] = (unsigned)hit;
                }
            }
        }
        if (wide && !long_rows)
            sweep_publish_wg<WAVES>(a, f, S, wid, nout, it + 1u, home, st);
        else if (nout > 0)
            sweep_publish(a, f, L, nout, it + 1u, home, long_rows, st);
        if (!gang_barrier<WAVES>(a, f, g, S, t_start)) break;
    }
    return result;
}

// Control words of a new solve and the source's items in the first buffer, by
// `threads` threads of one workgroup.
__device__ __forceinline__ void sweep_seed(const SolveArgs& a, const SweepArgs& f, unsigned tid,
                                           unsigned threads) {
    BQ_GLOBAL SweepCtl* c = f.ctl;
    const long long C = 1ll << a.chunk_log;
    const long long deg = a.off[a.src + 1] - a.off[a.src];
    const unsigned nch = deg > C ? (unsigned)((deg + C - 1) >> a.chunk_log) : 0u;
    for (unsigned k = tid; k < nch; k += threads)
        f.chunk[k] = ((unsigned long long)k << 32) | (unsigned)a.src;
    if (tid < 3 * MAX_SEG)
        c->tail[tid / MAX_SEG][tid % MAX_SEG].v =
            tid == 0 ? (nch ? (unsigned long long)nch << 32 : 1ull) : 0ull;
    if (tid < 8) c->arrive[tid].v = 0ull;
    if (tid != 0) return;
    if (nch == 0) f.light[0] = (unsigned)a.src;
    c->root.v = 0ull;
    c->joined.v = 0ull;
    c->go.v = 0ull;
}

// Chunk items one buffer's segment holds at most: a row longer than C gives
// ceil(degree / C) <= 2 degree / C of them.
inline unsigned long long sweep_chunk_cap(long long m, unsigned chunk_log) {
    return 2ull * ((unsigned long long)m >> chunk_log) + 64ull;
}

// Memory of a sweep solve, carved from `base` (256-byte aligned): words, the
// light and chunk items of the two buffers, the stamps. Returns its size.
// f->longp is the caller's.
inline unsigned long long sweep_layout(char* base, int n, long long m, unsigned chunk_log, int nseg,
                                       SweepArgs* f) {
    unsigned long long at = 0;
    auto take = [&](unsigned long long bytes) {
        char* p = base + at;
        at += (bytes + 255ull) & ~255ull;
        return p;
    };
    const unsigned long long cl = (unsigned long long)n, cc = sweep_chunk_cap(m, chunk_log);
    SweepArgs t{};
    t.ctl = (decltype(t.ctl))take(sizeof(SweepCtl));
    t.light = (decltype(t.light))take(4ull * 2ull * (unsigned long long)nseg * cl);
    t.chunk = (decltype(t.chunk))take(8ull * 2ull * (unsigned long long)nseg * cc);
    t.stamp = (decltype(t.stamp))take(4ull * cl);
    t.cap_light = (unsigned)cl;
    t.cap_chunk = (unsigned)cc;
    if (f) *f = t;
    return at;
}

}  // namespace
