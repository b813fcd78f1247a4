// The strip form of the queue-driven Bellman-Ford, for meshes whose vertex ids
// follow the mesh (rows of it, space-filling orders): the same keys,
// relaxations and results as the other forms, with each workgroup of a gang the
// owner of a strip of consecutive vertices.
//
// A strip's keys live in its workgroup's LDS, and so does its queue. A step
// relaxes the queued vertices with labels below the lowest one plus max |w|
// (the others stay queued); the workgroups take no notice of each other's
// steps. An edge into another strip becomes a message: the candidate is
// min-ed into the target's key in memory, and if that key's q bit was clear
// the target's number goes to the ring of its owner, who clears q, reads the
// candidate and min-s it into the key in LDS. The solve ends when every owner
// is idle and as many messages have been taken as sent.
//
// Why: a mesh's solve is a chain of thousands of steps of a few hundred
// relaxations each, and what counts is the time of one. In sweeps of the whole
// gang (sssp_sweep.hpp) it is about 6 us (a barrier of all workgroups and a
// chain of memory round trips), in the asynchronous form about 9 us per vertex
// of the chain; here a step is two dependent loads (row, edges) and an LDS
// atomic, and only a chain's crossings between strips, one in tens or hundreds
// of steps, pay for memory atomics. Two waves of the workgroup do those, beside
// the step of the others. And labels can be taken in order at once: a
// 2048 x 2048 road mesh relaxes each edge 2.1 times in 4,500 steps (counted on
// the CPU), where sweeps in FIFO order relax it 51 times at a quarter of the
// size.
//
// Ids that do not follow the mesh make every edge a message; the first
// workgroup looks at a sample of rows and refuses such a graph, as it does one
// with a row too long for one wave, with many edges between the strips of a graph
// that is no mesh, or with too few workgroups to hold the keys, and the caller's
// other form solves it. The members are those that run when the solve starts, so no launch waits
// for good for workgroups that other launches keep from running.
//
// A set q bit. In LDS it says that the vertex is in the strip's list (or, beyond
// the list's length, that the step's `over` is set): a strip starts with the
// source's alone set, and the source in the list; later only the min that
// finds it clear and sets it puts the vertex in the list, and taking the vertex
// clears it. In memory it says that the vertex's number is in its owner's ring:
// the words start without it (the source's owner clears the source's before it
// relaxes anything, and no candidate exists earlier), and only messages write
// them until the solve is over. So neither array is ever filled from the other,
// at the start least of all: a member that copied its keys from memory after
// another's message got there would hold a set bit for a vertex that is in no
// list, take the message for old news, and never relax the vertex.
//
// Memory ordering: keys in memory, ring words and rings are read and written
// by agent-scope atomics; an entry is valid once its tag is the one of its
// position. The LDS words of one step are separated from the next step's by
// the workgroup's barrier.
#pragma once
#include <hip/hip_runtime.h>
#include <limits.h>

#include "host_common.hpp"
#include "sssp_device.hpp"

namespace {

constexpr int STRIP_WG = 768;
constexpr int STRIP_WAVES = STRIP_WG / 64;
constexpr unsigned STRIP_WORKERS = 8;  // waves that relax; then one that stores
                                       // parents, one that walks on them or looks
                                       // for the end, one that sends, one that
                                       // receives
constexpr unsigned STRIP_MAX_N = 16384;     // vertices of a strip: 128 KiB of keys
constexpr unsigned STRIP_MAX_MEMBERS = 256;
constexpr unsigned STRIP_N = 8192;  // vertices of a strip by default, see strip_members
constexpr unsigned STRIP_LIST = 4096;       // queued vertices; beyond, a step looks at all keys
constexpr unsigned STRIP_OUT = 512;         // messages of a step; beyond, sent at once
// From this step on (a 2048 x 2048 road mesh takes a sixth of that) the walk for a
// negative cycle goes on in the steps in which the strip has nothing to do: on a
// cycle through many strips that is most of them, and with moves in busy steps
// alone one of 200,000 vertices took 17 s and one of 300,000, found after 1.1 s
// now, the whole of the solve's 20.
constexpr unsigned STRIP_WALK_IDLE = 1u << 16;
constexpr unsigned STRIP_ID_BITS = 14;      // of a ring entry; the rest is its tag
constexpr unsigned long long STRIP_REFUSED = ~0ull;
constexpr unsigned long long STRIP_STOP = 1ull << 63;    // in a tail word
constexpr unsigned long long STRIP_ACTIVE = 1ull << 63;  // in a state word
static_assert(STRIP_MAX_N == 1u << STRIP_ID_BITS, "a ring entry holds any vertex of a strip");

struct alignas(64) StripWord {
    unsigned long long v;
    unsigned long long pad[7];
};

struct StripCtl {
    StripWord joined;                    // workgroups that have asked to take part
    StripWord go;                        // 0, then the members, or STRIP_REFUSED
    StripWord tail[STRIP_MAX_MEMBERS];   // messages ever sent to a member; STRIP_STOP
    StripWord state[STRIP_MAX_MEMBERS];  // STRIP_ACTIVE, or sent << 32 | taken of an idle one
};

struct StripArgs {
    BQ_GLOBAL StripCtl* ctl;   // null: no strip form
    BQ_GLOBAL unsigned* mail;  // [strip_mail_words(n)] the members' rings, one after another
    BQ_GLOBAL unsigned* par;   // [n] parents of vertices when last relaxed, for the walks
    BQ_GLOBAL const unsigned* longp;  // per weight-range partial: longest row (note_row)
    unsigned max_row;          // longest row that it takes
    unsigned max_cross;        // edges between strips, of 1,024, that it takes where
                               // neighbourhoods grow fast
    unsigned want;             // members at most
};

struct alignas(16) StripStep {
    unsigned cnt;   // entries of the step's list
    unsigned over;  // whether vertices are queued that are not in the list
    unsigned nout;  // messages to send
    unsigned busy;  // whether messages are on their way through the last two waves
};

struct StripLds {
    long long key[STRIP_MAX_N];
    long long out_c[2][STRIP_OUT];
    unsigned out_v[2][STRIP_OUT];
    unsigned short list[2][STRIP_LIST];
    long long lo[3];   // words of a step by its number mod 3: lowest queued label,
    StripStep w[3];    // and the others
    unsigned sent;
    unsigned stop;       // number of the last step, plus one
    unsigned long long go;
    unsigned rank;
    // the first workgroup's sample: edges, those beyond the next strip and those
    // out of their own, the longest row; and what its probes found (strip_probe)
    unsigned rows, far, cross, lrow, ring4, ring5, dense;
    int wr[16][2];
    unsigned long long stats[bq::ST_N];
};

// Workgroups of a solve: one per STRIP_N vertices, at most `most`, but as many as
// the keys need. Road meshes with a strip per 2,048 / 4,096 / 8,192 vertices:
// 256 x 256 1.53 / 1.39 / 1.44 ms, 512 x 512 3.61 / 3.00 / 2.98, 1024 x 1024 7.4 /
// 7.4 / 6.1.
inline unsigned strip_members(long long n, long long most) {
    const long long w = n / STRIP_N < most ? n / STRIP_N : most;
    const long long need = (n + STRIP_MAX_N - 1) / STRIP_MAX_N;
    return (unsigned)(w < need ? need : w);
}

__host__ __device__ inline unsigned long long strip_mail_words(unsigned long long n) {
    return 2ull * (n + STRIP_MAX_MEMBERS);
}

// Memory of a strip solve, carved from `base` (256-byte aligned). Returns its
// size.
inline unsigned long long strip_layout(char* base, int n, StripArgs* p) {
    unsigned long long at = 0;
    auto take = [&](unsigned long long bytes) {
        char* q = base + at;
        at += (bytes + 255ull) & ~255ull;
        return q;
    };
    StripArgs t{};
    t.ctl = (decltype(t.ctl))take(sizeof(StripCtl));
    t.mail = (decltype(t.mail))take(4ull * strip_mail_words((unsigned long long)n));
    t.par = (decltype(t.par))take(4ull * (unsigned long long)n);
    if (p) *p = t;
    return at;
}

// Whether a graph may be one for strips on `workgroups` of them: short rows, keys
// that fit their LDS, and edges for more than one vertex in 16 (1M vertices with
// 10,000 edges 71 us without the strips' words to clear, 86 with).
inline bool strip_shape(long long n, long long m, long long workgroups) {
    return bqh::short_rows(n, m) && 16 * m >= n && n <= workgroups * (long long)STRIP_MAX_N;
}

// Longest row that strips take, where the sweeps solve the query otherwise, and
// where the queue solver does. One wave relaxes a row, and beyond its strip each
// edge is a message (25 ns an edge); and a row that reaches much of the graph
// leaves no long chain, which is what strips are for. Road meshes of n vertices
// with a row of L edges spread over them, ms in strips / in sweeps / by the queue
// solver: n = 90,000, L = 500 0.44 / 0.46 / 3.2, 2,000 0.44 / 0.30 / 3.2, 22,000
// 0.77 / 0.21 / 3.0, 90,000 2.3 / 0.21 / 3.2; 1M, 2,000 0.65 / 1.02 / 2.1, 8,000 0.69
// / 0.67 / 1.9, 64,000 1.86 / 0.50 / 1.9, 128,000 3.4 / 0.49 / 1.9; 4M, 8,000 1.34 /
// 2.1 / 5.2, 32,000 1.81 / 1.57 / 4.7, 128,000 4.1 / 1.3 / 4.4.
inline unsigned strip_row_sweeps(long long n) { return (unsigned)(n / 128); }
constexpr unsigned STRIP_ROW_QUEUE = 65536;

// Edges out of a strip, of 1,024, that strips take from a graph whose
// neighbourhoods grow like a tree's and not like a mesh's (strip_probe): there a
// step holds thousands of vertices, few strips are busy at a time, and a good
// part of a strip's work is messages. Such graphs of n vertices with edges to
// random ids within K, of out-degree g, ms in strips / in sweeps / by the queue
// solver: n = 1M, g = 3, K = 300 (2 % of the edges leave the strip) 19 / 59 / 28,
// 1,000 (6 %) 18 / 18 / 8.7, 2,000 (12 %) 21 / 9.9 / 4.6, 8,000 21 / 2.5 / 1.9; g = 5.5,
// 300 39 / 81 / 34, 1,000 39 / 28 / 11; n = 30,000, g = 5.5, 2,000 (7 %) 1.6 / 0.38 /
// 2.1, 4,000 (13 %) 1.8 / 0.32 / 2.0, 8,000 (27 %) 3.1 / 0.29 / 2.0. A 256 x 4,096
// mesh, 25 % of whose edges leave their strip, takes 19 / 108 / 51. From 3/8 on
// strips lose on all.
constexpr unsigned STRIP_CROSS_SWEEPS = 82;
inline unsigned strip_cross_queue(long long n) { return n < 65536 ? 146u : 16u; }

// Words of a new solve, by threads tid of `threads`: rings and parents of
// vertices [v0, v1); with `first` the control words and the rings' rest.
__device__ __forceinline__ void strip_seed(const StripArgs& p, long long n, long long v0,
                                           long long v1, bool first, long long tid,
                                           long long threads) {
    for (long long v = v0 + tid; v < v1; v += threads) {
        p.mail[2 * v] = 0u;
        p.mail[2 * v + 1] = 0u;
        p.par[v] = ~0u;
    }
    if (!first) return;
    for (long long i = tid; i < (long long)STRIP_MAX_MEMBERS; i += threads) {
        p.mail[2 * n + 2 * i] = 0u;
        p.mail[2 * n + 2 * i + 1] = 0u;
        p.ctl->tail[i].v = 0ull;
        p.ctl->state[i].v = STRIP_ACTIVE;
    }
    if (tid == 0) {
        p.ctl->joined.v = 0ull;
        p.ctl->go.v = 0ull;
    }
}

template <int CTRL, int ROWS>
__device__ __forceinline__ long long min_dpp(long long x) {
    const int l = (int)x, h = (int)(x >> 32);
    const int yl = __builtin_amdgcn_update_dpp(l, l, CTRL, ROWS, 0xf, false);
    const int yh = __builtin_amdgcn_update_dpp(h, h, CTRL, ROWS, 0xf, false);
    const long long y = (long long)(((unsigned long long)(unsigned)yh << 32) | (unsigned)yl);
    return y < x ? y : x;
}

// the wave's minimum, in lane 63
__device__ __forceinline__ long long wave_min(long long x) {
    x = min_dpp<0x111, 0xf>(x);  // row_shr:1, 2, 4, 8
    x = min_dpp<0x112, 0xf>(x);
    x = min_dpp<0x114, 0xf>(x);
    x = min_dpp<0x118, 0xf>(x);
    x = min_dpp<0x142, 0xa>(x);  // row_bcast:15, 31
    return min_dpp<0x143, 0xc>(x);
}

// the value of the first lane of each four
__device__ __forceinline__ long long quad_first(long long x) {
    const int l = __builtin_amdgcn_update_dpp(0, (int)x, 0x00, 0xf, 0xf, false);
    const int h = __builtin_amdgcn_update_dpp(0, (int)(x >> 32), 0x00, 0xf, 0xf, false);
    return (long long)(((unsigned long long)(unsigned)h << 32) | (unsigned)l);
}

// One wave: every member's next look at its ring ends its solve.
__device__ __forceinline__ void strip_stop_all(const StripArgs& p, unsigned members) {
    for (unsigned r = bq::lane_id(); r < members; r += 64)
        __hip_atomic_fetch_or(&p.ctl->tail[r].v, STRIP_STOP, __ATOMIC_RELAXED,
                              __HIP_MEMORY_SCOPE_AGENT);
}

// Vertices 4 and 5 edges away from a sample vertex of this wave, added to S.ring4
// and S.ring5 (8 edges of a row at most), or S.dense, if they are too many for
// the wave's part of the keys' array, which is not in use yet. The fifth ring of a
// plane mesh has 1.2 times the fourth's vertices, of a 3-dimensional grid 1.5, of
// random ids within a band twice and more until the band is full. Five pairs
// of dependent loads, 10 us.
__device__ __forceinline__ void strip_probe(const SolveArgs& a, StripLds& S, unsigned wid) {
    constexpr unsigned SET = 1024, LIST = 512;
    static_assert(sizeof(S.key) >= STRIP_WAVES * (SET + 2 * LIST) * sizeof(unsigned), "");
    const unsigned lane = (unsigned)bq::lane_id();
    unsigned* set = (unsigned*)S.key + wid * (SET + 2 * LIST);
    unsigned* cur = set + SET;
    unsigned* nxt = cur + LIST;
    const auto insert = [&](unsigned v) -> bool {  // whether it is new; never full
        unsigned h = (v * 2654435761u) >> 22;
        for (;;) {
            const unsigned old = atomicCAS(&set[h], ~0u, v);
            if (old == ~0u) return true;
            if (old == v) return false;
            h = (h + 1u) & (SET - 1u);
        }
    };
    for (unsigned i = lane; i < SET; i += 64) set[i] = ~0u;
    __builtin_amdgcn_wave_barrier();
    if (lane == 0) {
        cur[0] = (unsigned)((unsigned long long)a.n * (2u * wid + 1u) / (2u * STRIP_WAVES));
        insert(cur[0]);
    }
    __builtin_amdgcn_wave_barrier();
    unsigned nc = 1, seen = 1, ring[2] = {0u, 0u};
    bool dense = false;
    for (int hop = 1; hop <= 5 && !dense; ++hop) {
        unsigned nn = 0;
        for (unsigned b = 0; b < nc && !dense; b += 64) {
            long long e = 0, e1 = 0;
            if (b + lane < nc) {
                const unsigned u = cur[b + lane];
                e = a.off[u];
                e1 = a.off[u + 1];
            }
            int c[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) c[j] = e + j < e1 ? a.col[e + j] : -1;
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                if (seen + 64u > SET - 64u || nn + 64u > LIST) dense = true;  // wave-uniform
                if (!dense) {
                    const bool fresh = c[j] >= 0 && insert((unsigned)c[j]);
                    const unsigned long long m = bq::ballot(fresh);
                    if (fresh) nxt[nn + (unsigned)bq::rank_in(m)] = (unsigned)c[j];
                    nn += (unsigned)__popcll(m);
                    seen += (unsigned)__popcll(m);
                }
            }
        }
        __builtin_amdgcn_wave_barrier();
        unsigned* t = cur;
        cur = nxt;
        nxt = t;
        nc = nn;
        if (hop >= 4) ring[hop - 4] = nn;
    }
    if (lane != 0) return;
    if (dense) atomicOr(&S.dense, 1u);
    atomicAdd(&S.ring4, ring[0]);
    atomicAdd(&S.ring5, ring[1]);
}

// The solve of one query by up to p.want workgroups that call it with the same
// arguments (STRIP_WG threads each or more, `S` in LDS). Returns 1 when the query was
// solved or stopped by those that took it, 0 when it is left to another form.
__device__ __forceinline__ int strip_instance(const SolveArgs& a, const StripArgs& p, StripLds& S,
                                              WaveStats& st) {
    const unsigned lane = (unsigned)bq::lane_id();
    const unsigned wid = (unsigned)bq::bcast32(threadIdx.x >> 6);
    const unsigned shift = a.shift;
    const unsigned none = (1u << (shift - 1u)) - 1u;
    BQ_GLOBAL StripCtl* ctl = p.ctl;
    const unsigned long long t_start = bq::ld_rlx(&a.q.ctrl->aux[4].v);

    // ---- members ------------------------------------------------------------
    if (threadIdx.x == 0) {
        S.rank = (unsigned)bq::add_rlx(&ctl->joined.v, 1ull);
        S.rows = S.far = S.cross = S.lrow = S.ring4 = S.ring5 = S.dense = 0u;
        if (S.rank == 0) {
            // The others get 10 us; as many as hold the keys get up to 20 us each,
            // which other launches on the chip may take to end, times 1 to 4,
            // so that two solves that share the chip do not give up together.
            const unsigned long long t0 = bq::now_ticks();
            const unsigned long long need =
                ((unsigned long long)a.n + STRIP_MAX_N - 1ull) / STRIP_MAX_N;
            const unsigned long long most = 1000ull + 2000ull * need * (1ull + (t_start & 3ull));
            unsigned long long j, t;
            do {
                j = bq::ld_rlx(&ctl->joined.v);
                t = bq::now_ticks();
            } while (j < p.want && t - t0 < (j < need ? most : 1000ull) &&
                     t - t_start < a.deadline);
            S.go = j < p.want ? j : p.want;
        }
    }
    __syncthreads();
    const unsigned rank = S.rank;
    if (rank == 0) {
        const unsigned m0 = (unsigned)S.go;
        const unsigned per0 = ((unsigned)a.n + m0 - 1u) / m0;
        // a row per thread: edges that lead further than into the next strip
        const unsigned v =
            (unsigned)((unsigned long long)a.n * threadIdx.x / blockDim.x);
        long long e = a.off[v], e1 = a.off[v + 1];
        unsigned rows = 0, far = 0, cross = 0;
        for (int k = 0; k < 8 && e < e1; ++k, ++e) {
            const long long d = (long long)a.col[e] - (long long)v;
            ++rows;
            far += (d < 0 ? -d : d) > (long long)per0;
            cross += (unsigned)a.col[e] / per0 != v / per0;
        }
        unsigned lrow = 0;
        const int parts = (int)bq::ld_rlx(&a.q.ctrl->aux[0].v);
        for (int i = (int)threadIdx.x; i < parts; i += (int)blockDim.x)
            lrow = p.longp[i] > lrow ? p.longp[i] : lrow;
        atomicAdd(&S.rows, rows);
        atomicAdd(&S.far, far);
        atomicAdd(&S.cross, cross);
        atomicMax(&S.lrow, lrow);
        __syncthreads();
        bool ok = per0 <= STRIP_MAX_N && S.far * 16u <= S.rows && S.lrow <= p.max_row &&
                  S.cross * 8u <= S.rows * 3u;
        if (ok && __builtin_expect(S.cross * 1024u > S.rows * p.max_cross, 0)) {
            if (wid < (unsigned)STRIP_WAVES) strip_probe(a, S, wid);
            __syncthreads();
            ok = S.dense == 0u && S.ring5 * 10u <= S.ring4 * 17u;
        }
        if (threadIdx.x == 0) {
            S.go = ok ? (unsigned long long)m0 : STRIP_REFUSED;
            bq::st_rlx(&ctl->go.v, S.go);
        }
    } else if (threadIdx.x == 0) {
        // the first workgroup runs, and decides at the latest when its wait
        // above ends: 10 us, or until the keys' workgroups are there 20 us each
        // times up to 4 (20 ms for 256), within the solve's deadline
        unsigned long long go;
        do go = bq::ld_rlx(&ctl->go.v);
        while (go == 0ull);
        S.go = go;
    }
    __syncthreads();
    const unsigned long long go = S.go;
    if (go == STRIP_REFUSED) return 0;
    const unsigned members = (unsigned)go;
    if (rank >= members) return 1;  // solved by others

    // ---- weight range -------------------------------------------------------
    long long lbound, delta;
    {
        const int parts = (int)bq::ld_rlx(&a.q.ctrl->aux[0].v);
        int lo = INT_MAX, hi = INT_MIN;
        for (int i = (int)threadIdx.x; i < parts; i += (int)blockDim.x) {
            const int x = a.wrange[2 * i], y = a.wrange[2 * i + 1];
            lo = x < lo ? x : lo;
            hi = y > hi ? y : hi;
        }
        for (int off = 32; off > 0; off >>= 1) {
            const int x = __shfl_xor(lo, off, 64), y = __shfl_xor(hi, off, 64);
            lo = x < lo ? x : lo;
            hi = y > hi ? y : hi;
        }
        if (lane == 0) {
            S.wr[wid][0] = lo;
            S.wr[wid][1] = hi;
        }
        __syncthreads();
        long long wmin = INT_MAX, wmax = INT_MIN;
        for (unsigned i = 0; i < blockDim.x >> 6; ++i) {
            wmin = S.wr[i][0] < wmin ? S.wr[i][0] : wmin;
            wmax = S.wr[i][1] > wmax ? S.wr[i][1] : wmax;
        }
        long long maxabs = 0;
        if (a.m > 0) {
            maxabs = wmax > -wmin ? wmax : -wmin;
            if (maxabs < 0) maxabs = -maxabs;
        }
        // the packing precondition of all forms; every member sees the same
        // range, and the first one to leave stops nobody else
        if ((double)a.n * (double)maxabs >= (double)(1ull << (62u - shift))) {
            if (threadIdx.x == 0) bq::raise_error(a.q, bq::ERR_RANGE);
            return 1;
        }
        lbound = (long long)(a.n - 1) * (wmin < 0 ? wmin : 0ll);
        // Labels below the lowest queued one plus max |w| are relaxed in one
        // step: with half of that the steps of a 2048 x 2048 road mesh are 1.3
        // times as many, with twice that 1.3 % fewer and the relaxations 2.9
        // times as many (counted on the CPU).
        delta = maxabs > 0 ? maxabs : 1;
    }

    // ---- the strip ----------------------------------------------------------
    const unsigned per = ((unsigned)a.n + members - 1u) / members;
    unsigned rlog = 0;
    while ((1u << rlog) < per) ++rlog;
    const unsigned rmask = (1u << rlog) - 1u;
    const unsigned base = rank * per;
    const unsigned cnt = base < (unsigned)a.n
                             ? ((unsigned)a.n - base < per ? (unsigned)a.n - base : per)
                             : 0u;
    BQ_GLOBAL const unsigned* ring = p.mail + ((unsigned long long)rank << rlog);
    // The keys of a new solve are known, so they are not read from memory: other
    // members may be under way, and their first messages be in memory already.
    for (unsigned i = threadIdx.x; i < cnt; i += blockDim.x)
        S.key[i] = base + i == (unsigned)a.src ? pack_key(0, none, shift) : KEY_INF;
    if (threadIdx.x < 3) {
        S.lo[threadIdx.x] = LLONG_MAX;
        S.w[threadIdx.x] = StripStep{};
    }
    if (threadIdx.x == 0) {
        S.sent = 0u;
        S.stop = 0u;
    }
    // edges are numbered in 32 bits (fewer than 6 per vertex), and the loads take
    // a scalar base and a 32-bit offset
    const auto edge_of = [&](unsigned v) {
        return *(BQ_GLOBAL const unsigned*)((BQ_GLOBAL const char*)a.off + v * 8u);
    };
    const auto col_of = [&](unsigned e) {
        return *(BQ_GLOBAL const int*)((BQ_GLOBAL const char*)a.col + e * 4u);
    };
    const auto w_of = [&](unsigned e) {
        return *(BQ_GLOBAL const int*)((BQ_GLOBAL const char*)a.w + e * 4u);
    };
    // The strip's rows once through the caches: a step waits for the slowest
    // of its lanes, and some lane's line would always be a first touch.
    unsigned mix = 0;
    if (cnt != 0u) {
        const unsigned e1 = edge_of(base + cnt);
        for (unsigned v = threadIdx.x; v < cnt; v += blockDim.x) mix ^= edge_of(base + v);
        for (unsigned e = edge_of(base) + threadIdx.x * 16u; e < e1; e += blockDim.x * 16u)
            mix ^= (unsigned)(col_of(e) ^ w_of(e));
    }
    if (__all(mix == 0x9E3779B9u)) S.rows = mix;  // keeps the loads
    __syncthreads();
    if (threadIdx.x == 0 && (unsigned)a.src - base < cnt) {
        // the source is queued here (q is set in its key in LDS), and messages
        // to it find q clear
        S.list[0][0] = (unsigned short)((unsigned)a.src - base);
        S.w[0].cnt = 1u;
        S.lo[0] = 0;
        __hip_atomic_fetch_and(&a.key[a.src], ~1ll, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    }
    __syncthreads();

    // The waves of the four roles run loops of their own, a step each between
    // two barriers; what a sender or receiver has in flight stays so across
    // the barrier.
    const long long labels = -(1ll << shift);  // a key's label bits
    unsigned step = 0, cur = 0, nx = 1, b0 = 0, b1 = 1;
    StripStep now{};
    bool pending = false;
    bool flagged = false;      // marking mode: this wave already raised negcycle
    long long lo = LLONG_MAX;  // lowest label this lane queues
    bool neg = false;
    const auto begin = [&]() {
        if (threadIdx.x == 0) {
            const unsigned z = 3u - cur - nx;  // last read in the step before
            S.lo[z] = LLONG_MAX;
            S.w[z] = StripStep{};
        }
        now = S.w[cur];
        now.nout = now.nout < STRIP_OUT ? now.nout : STRIP_OUT;
        pending = (now.cnt | now.over | now.nout | now.busy) != 0u;
    };
    // whether there is another step
    const auto end = [&]() -> bool {
        if (__any(neg)) {
            if (!flagged) {
                if (lane == 0) bq::st_rlx(&a.q.ctrl->negcycle.v, 1ull);
                if (!a.neginf) {
                    if (lane == 0) bq::st_rlx(&a.q.ctrl->abort.v, 1ull);
                    strip_stop_all(p, members);
                }
            }
            flagged = true;
            neg = false;
        }
        if (__any(lo != LLONG_MAX)) {
            // (64 lanes that min into one LDS word take 2,000 cycles)
            lo = wave_min(lo);
            if (lane == 63u)
                __hip_atomic_fetch_min(&S.lo[nx], lo, __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_WORKGROUP);
            lo = LLONG_MAX;
        }
        ++step;
        cur = nx;
        nx = nx == 2u ? 0u : nx + 1u;
        b0 = b1;
        b1 ^= 1u;
        __syncthreads();
        // a stop written in the step after this one is seen at its end
        const unsigned stop = S.stop;
        return stop == 0u || stop > step;
    };
    // queue vertex li of the strip, label d, for the next step; their number
    const auto queue = [&](bool push, unsigned li, long long d) -> unsigned long long {
        const unsigned long long pm = bq::ballot(push);
        if (pm == 0ull) return 0ull;
        unsigned at = 0;
        if (lane == 0) at = atomicAdd(&S.w[nx].cnt, (unsigned)__popcll(pm));
        at = (unsigned)bq::bcast32((int)at) + (unsigned)bq::rank_in(pm);
        if (push) {
            if (at < STRIP_LIST) S.list[b1][at] = (unsigned short)li;
            else S.w[nx].over = 1u;
            lo = d < lo ? d : lo;
        }
        return (unsigned long long)__popcll(pm);
    };
    // message to the owner of vertex c
    const auto send = [&](bool live, unsigned c, long long cand) {
        bool push = false;
        if (live) {
            const long long old = __hip_atomic_fetch_min(&a.key[c], cand, __ATOMIC_RELAXED,
                                                         __HIP_MEMORY_SCOPE_AGENT);
            push = cand < old && (old & 1ll) == 0;
        }
        const unsigned long long pm = bq::ballot(push);
        if (pm == 0ull) return;
        if (push) {
            const unsigned o = c / per;
            const unsigned at = (unsigned)bq::add_rlx(&ctl->tail[o].v, 1ull);
            bq::st_rlx(&p.mail[((unsigned long long)o << rlog) + (at & rmask)],
                       ((((at >> rlog) + 1u) << STRIP_ID_BITS) | (c - o * per)));
        }
        if (lane == 0) atomicAdd(&S.sent, (unsigned)__popcll(pm));
    };
    const auto post = [&](bool live, unsigned c, long long cand) {
        const unsigned long long pm = bq::ballot(live);
        if (pm == 0ull) return;
        unsigned at = 0;
        if (lane == 0) at = atomicAdd(&S.w[nx].nout, (unsigned)__popcll(pm));
        at = (unsigned)bq::bcast32((int)at) + (unsigned)bq::rank_in(pm);
        if (live && at < STRIP_OUT) {
            S.out_v[b1][at] = c;
            S.out_c[b1][at] = cand;
        }
        if (__builtin_expect(__any(live && at >= STRIP_OUT), 0)) send(live && at >= STRIP_OUT, c, cand);
    };
    // candidate into key li of the strip
    const auto lower = [&](bool live, unsigned li, long long cand, long long cd) {
        long long old = LLONG_MIN;
        if (live)
            old = __hip_atomic_fetch_min(&S.key[li], cand, __ATOMIC_RELAXED,
                                         __HIP_MEMORY_SCOPE_WORKGROUP);
        const bool won = live && cand < old;
        const bool dropped = won && ((cand ^ old) & labels) != 0;
        st.impr += dropped;
        neg |= dropped && cd < lbound;
        st.push += queue(won && (old & 1ll) == 0, li, cd);
    };
    // up to K edges per lane from vertex pu with label du; their queueing takes
    // one add to the list's count per wave, their messages another
    const auto relax = [&](const auto& live, const auto& c, const auto& w, long long du,
                           unsigned pu) {
        constexpr int K = (int)(sizeof(c) / sizeof(c[0]));
        long long cand[K], cd[K], old[K];
        bool mine[K], push[K], cross[K];
        unsigned npush = 0, ncross = 0;  // of the wave, in lane order within an edge
        unsigned rank_p[K], rank_c[K];
#pragma unroll
        for (int j = 0; j < K; ++j) {
            cd[j] = du + (long long)w[j];
            cand[j] = pack_key(cd[j], pu, shift);
            // marking mode: below the certain lower bound (or from a
            // minus-infinity source) a negative cycle reaches the target
            if (a.neginf && cd[j] < lbound) cand[j] = KEY_NEG;
            mine[j] = live[j] && (unsigned)c[j] - base < cnt;
            cross[j] = live[j] && !mine[j];
            old[j] = LLONG_MIN;
            if (mine[j])
                old[j] = __hip_atomic_fetch_min(&S.key[(unsigned)c[j] - base], cand[j],
                                                __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            st.relax += (unsigned long long)__popcll(bq::ballot(live[j]));
            const unsigned long long cm = bq::ballot(cross[j]);
            rank_c[j] = ncross + (unsigned)bq::rank_in(cm);
            ncross += (unsigned)__popcll(cm);
        }
#pragma unroll
        for (int j = 0; j < K; ++j) {
            const bool won = mine[j] && cand[j] < old[j];
            const bool dropped = won && ((cand[j] ^ old[j]) & labels) != 0;
            st.impr += dropped;
            neg |= dropped && cd[j] < lbound;
            push[j] = won && (old[j] & 1ll) == 0;
            const unsigned long long pm = bq::ballot(push[j]);
            rank_p[j] = npush + (unsigned)bq::rank_in(pm);
            npush += (unsigned)__popcll(pm);
        }
        st.push += npush;
        if ((npush | ncross) == 0u) return;
        unsigned at_p = 0, at_c = 0;
        if (lane == 0) {
            if (npush != 0u) at_p = atomicAdd(&S.w[nx].cnt, npush);
            if (ncross != 0u) at_c = atomicAdd(&S.w[nx].nout, ncross);
        }
        at_p = bq::bcast32(at_p);
        at_c = bq::bcast32(at_c);
#pragma unroll
        for (int j = 0; j < K; ++j) {
            if (push[j]) {
                const unsigned at = at_p + rank_p[j];
                if (at < STRIP_LIST) S.list[b1][at] = (unsigned short)((unsigned)c[j] - base);
                else S.w[nx].over = 1u;
                lo = cd[j] < lo ? cd[j] : lo;
            }
            if (cross[j] && at_c + rank_c[j] < STRIP_OUT) {
                S.out_v[b1][at_c + rank_c[j]] = (unsigned)c[j];
                S.out_c[b1][at_c + rank_c[j]] = cand[j];
            }
        }
        // rare, and kept out of the loop's way (2048 x 2048 road mesh 13.4 -> 13.0 ms)
        if (__builtin_expect(at_c + ncross > STRIP_OUT, 0))
#pragma unroll
            for (int j = 0; j < K; ++j)
                send(cross[j] && at_c + rank_c[j] >= STRIP_OUT, (unsigned)c[j], cand[j]);
    };

    if (wid < STRIP_WORKERS) {
        // ---- relax ----------------------------------------------------------
        do {
            begin();
            const bool scan = now.over != 0u;
            const unsigned items = scan ? cnt : (now.cnt < STRIP_LIST ? now.cnt : STRIP_LIST);
            const long long T = items != 0u ? S.lo[cur] + delta : 0ll;
            // A step of few items gives each 4 lanes, one edge per lane at a
            // time; else a lane takes an item and up to 8 edges. The rest of
            // longer rows is scanned by the whole wave.
            const bool few = items <= STRIP_WORKERS * 32u;
            const unsigned sub = few ? lane & 3u : 0u, ipw = few ? 16u : 64u;
            for (unsigned i0 = wid * ipw; i0 < items; i0 += STRIP_WORKERS * ipw) {
                const unsigned i = i0 + (few ? lane >> 2 : lane);
                unsigned v = 0, e0 = 0, e1 = 0;
                long long k = 0, du = 0;
                if (i < items) {
                    v = scan ? i : (unsigned)S.list[b0][i];
                    // read before the label tells whether they are needed
                    e0 = edge_of(base + v);
                    e1 = edge_of(base + v + 1u);
                    k = S.key[v];
                }
                const bool live = (k & 1ll) != 0;  // still queued
                const bool near = live && (k >> shift) < T;
                if (near && sub == 0u)
                    k = __hip_atomic_fetch_and(&S.key[v], ~1ll, __ATOMIC_RELAXED,
                                               __HIP_MEMORY_SCOPE_WORKGROUP);
                if (few) k = quad_first(k);
                if (!near) e1 = e0;
                if (__any(live && !near)) queue(live && !near && sub == 0u, v, k >> shift);
                du = k >> shift;
                st.deq += (unsigned long long)__popcll(bq::ballot(near && sub == 0u));
                if (few) {
                    for (unsigned r = sub; r < 8u && __any(e0 + r < e1); r += 4u) {
                        const unsigned e = e0 + r;
                        const bool in[1] = {e < e1};
                        const int c[1] = {in[0] ? col_of(e) : 0}, w[1] = {in[0] ? w_of(e) : 0};
                        relax(in, c, w, du, base + v);
                    }
                } else {
                    bool in[2][4];
                    int c[2][4], w[2][4];
#pragma unroll
                    for (unsigned j = 0; j < 8; ++j) {
                        in[j / 4][j % 4] = e0 + j < e1;
                        c[j / 4][j % 4] = e0 + j < e1 ? col_of(e0 + j) : 0;
                        w[j / 4][j % 4] = e0 + j < e1 ? w_of(e0 + j) : 0;
                    }
                    relax(in[0], c[0], w[0], du, base + v);
                    if (__any(in[1][0])) relax(in[1], c[1], w[1], du, base + v);
                }
                unsigned long long rest = bq::ballot(e1 - e0 > 8u && sub == 0u);
                while (rest != 0ull) {
                    const int l = __ffsll((unsigned long long)rest) - 1;
                    rest &= rest - 1ull;
                    const unsigned s = (unsigned)__shfl((int)e0, l, 64) + 8u;
                    const unsigned t = (unsigned)__shfl((int)e1, l, 64);
                    const long long d = __shfl(du, l, 64);
                    const unsigned u = base + (unsigned)__shfl((int)v, l, 64);
                    for (unsigned x = s; x < t; x += 256u) {
                        bool in[4];
                        int c[4], w[4];
#pragma unroll
                        for (unsigned j = 0; j < 4; ++j) {
                            const unsigned e = x + 64u * j + lane;
                            in[j] = e < t;
                            c[j] = in[j] ? col_of(e) : 0;
                            w[j] = in[j] ? w_of(e) : 0;
                        }
                        relax(in, c, w, d, u);
                    }
                }
            }
        } while (end());
    } else if (wid == STRIP_WORKERS) {
        // ---- parents of the step's vertices, for the walks ------------------
        // by a wave that waits for nothing: a worker's loads would wait for its
        // stores, which take longer
        do {
            begin();
            const bool scan = now.over != 0u;
            const unsigned items = scan ? cnt : (now.cnt < STRIP_LIST ? now.cnt : STRIP_LIST);
            for (unsigned i = lane; i < items; i += 64u) {
                const unsigned v = scan ? i : (unsigned)S.list[b0][i];
                const long long k = S.key[v];
                // (in a scan the q bit tells nothing: the workers, eight times as
                // fast, have cleared it)
                if (!scan || k != KEY_INF)
                    bq::st_rlx(&p.par[base + v],
                               is_neg_key(k) ? none : (unsigned)((unsigned long long)k >> 1) & none);
            }
        } while (end());
    } else if (wid == STRIP_WORKERS + 1u) {
        // ---- look for the end, walk -----------------------------------------
        SweepWalk<false> walk{};
        const auto parent = [&](unsigned x) {
            const unsigned q = bq::ld_rlx(&p.par[x]);
            return q < (unsigned)a.n ? q : none;
        };
        unsigned long long seen[4] = {};  // the latest look at the state words
        bool was_end = false;
        do {
            begin();
            if (!pending && rank == 0) {
                // ---- the end: all idle, and nothing changed since the look
                // before (which ended before this one began), and no message
                // on its way
                bool same = true, idle = true;
                unsigned sent = 0, got = 0;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const unsigned r = (unsigned)j * 64u + lane;
                    if (r < members) {
                        const unsigned long long x = bq::ld_rlx(&ctl->state[r].v);
                        idle = idle && (x & STRIP_ACTIVE) == 0ull;
                        same = same && x == seen[j];
                        seen[j] = x;
                        sent += (unsigned)(x >> 32);
                        got += (unsigned)x;
                    }
                }
                for (int off = 32; off > 0; off >>= 1) {
                    sent += __shfl_xor(sent, off, 64);
                    got += __shfl_xor(got, off, 64);
                }
                const bool end = __all(idle) && ((sent ^ got) & 0x7FFFFFFFu) == 0u;
                if (end && was_end && __all(same)) strip_stop_all(p, members);
                was_end = end;
            } else if (pending && step >= SWEEP_WALK_FROM) {
                // ---- negative cycles: some moves on the parents a step ------
                int hit = -1;
                if (!walk.on && now.cnt != 0u) {  // (the list's start holds whatever is over)
                    const unsigned q = now.cnt < STRIP_LIST ? now.cnt : STRIP_LIST;
                    walk.start(base + (unsigned)bq::bcast32((int)S.list[b0][step % q]), parent);
                    ++st.walk;
                } else if (walk.on) {
                    // moves that the step's own work leaves time for
                    const unsigned more = now.cnt >> 7;
                    hit = walk.advance(a, parent, 1u + (more < 31u ? more : 31u));
                }
                if (hit >= 0) {
                    if (lane == 0) bq::st_rlx(&a.q.ctrl->negcycle.v, 1ull);
                    flagged = true;
                    if (!a.neginf) {
                        if (lane == 0) bq::st_rlx(&a.q.ctrl->abort.v, 1ull);
                        strip_stop_all(p, members);
                    } else {
                        // the cycle's vertex becomes minus infinity and spreads
                        // it through the queue like any lowered label
                        const bool mine = (unsigned)hit - base < cnt;
                        lower(lane == 0 && mine, (unsigned)hit - base, KEY_NEG, KEY_NEG >> shift);
                        post(lane == 0 && !mine, (unsigned)hit, KEY_NEG);
                    }
                }
            } else if (!pending && step >= STRIP_WALK_IDLE) {
                // what a walk that has closed shows is for a busy step: an idle
                // strip, whose state word says so, sends and queues nothing. (This
                // branch ahead of the busy steps' cost all steps 9 %.)
                walk.move(a, parent);
            }
        } while (end());
    } else if (wid == STRIP_WORKERS + 2u) {
        // ---- send: minimum, tail and entry of a message in a step each ------
        bool live0 = false, live1 = false;
        unsigned c0 = 0, c1 = 0, o1 = 0, at1 = 0;
        long long cand0 = 0, old0 = 0;
        do {
            begin();
            if (live1)
                bq::st_rlx(&p.mail[((unsigned long long)o1 << rlog) + (at1 & rmask)],
                           (((at1 >> rlog) + 1u) << STRIP_ID_BITS) | c1);
            live1 = live0 && cand0 < old0 && (old0 & 1ll) == 0;
            const unsigned long long pm = bq::ballot(live1);
            if (live1) {
                o1 = c0 / per;
                c1 = c0 - o1 * per;
                at1 = (unsigned)bq::add_rlx(&ctl->tail[o1].v, 1ull);
            }
            if (pm != 0ull && lane == 0) atomicAdd(&S.sent, (unsigned)__popcll(pm));
            live0 = lane < now.nout;
            if (live0) {
                c0 = S.out_v[b0][lane];
                cand0 = S.out_c[b0][lane];
                old0 = __hip_atomic_fetch_min(&a.key[c0], cand0, __ATOMIC_RELAXED,
                                              __HIP_MEMORY_SCOPE_AGENT);
            }
            for (unsigned i = 64; i < now.nout; i += 64) {
                const bool live = i + lane < now.nout;
                send(live, live ? S.out_v[b0][i + lane] : 0u, live ? S.out_c[b0][i + lane] : 0ll);
            }
            if ((now.nout != 0u || pm != 0ull) && lane == 0) S.w[nx].busy = 1u;
        } while (end());
    } else if (wid == STRIP_WORKERS + 3u) {
        // ---- receive: tail, entries and labels in a step each ---------------
        unsigned head = 0, taken = 0;  // messages taken and applied (mod 2^32)
        bool told_idle = false;        // the state word says idle
        unsigned n_entry = 0, n_label = 0, entry = 0, li = 0;
        long long label = 0;
        unsigned long long tail = bq::ld_rlx(&ctl->tail[rank].v);
        do {
            begin();
            if (n_label != 0u) {
                lower(lane < n_label, li, label | 1ll, label >> shift);
                taken += n_label;
                n_label = 0u;
            }
            if (n_entry != 0u) {
                const unsigned at = head + lane;
                const unsigned tag = ((at >> rlog) + 1u) << STRIP_ID_BITS;
                const unsigned long long ready =
                    bq::ballot(lane < n_entry && (entry & ~(STRIP_MAX_N - 1u)) == tag);
                n_label = ready == ~0ull ? 64u : (unsigned)__ffsll(~ready) - 1u;
                if (lane < n_label) {
                    li = entry & (STRIP_MAX_N - 1u);
                    label = __hip_atomic_fetch_and(&a.key[base + li], ~1ll, __ATOMIC_RELAXED,
                                                   __HIP_MEMORY_SCOPE_AGENT);
                }
                head += n_label;
                n_entry = 0u;
            }
            const unsigned long long t = bq::bcast64(tail);
            const unsigned avail = (unsigned)t - head;
            if (avail != 0u) {
                if (told_idle) {
                    // active again, and known to be before anything is sent
                    if (lane == 0) bq::st_rlx(&ctl->state[rank].v, STRIP_ACTIVE);
                    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                    told_idle = false;
                }
                n_entry = avail < 64u ? avail : 64u;
                if (lane < n_entry) entry = bq::ld_rlx(&ring[(head + lane) & rmask]);
            }
            tail = bq::ld_rlx(&ctl->tail[rank].v);
            if (n_entry != 0u || n_label != 0u) {
                if (lane == 0) S.w[nx].busy = 1u;
            } else if (!pending && !told_idle) {
                if (lane == 0)
                    bq::st_rlx(&ctl->state[rank].v,
                               ((unsigned long long)(S.sent & 0x7FFFFFFFu) << 32) | taken);
                told_idle = true;
            }
            bool stop = (t & STRIP_STOP) != 0ull;
            if ((step & 63u) == 0u && bq::now_ticks() - t_start > a.deadline) {
                if (lane == 0) bq::raise_error(a.q, bq::ERR_TIMEOUT);
                strip_stop_all(p, members);
                stop = true;
            }
            if (stop && lane == 0) S.stop = step + 1u;
        } while (end());
    } else {
        while (end()) {
        }
    }
    if (wid == 0u) st.batch += step;
    for (unsigned i = threadIdx.x; i < cnt; i += blockDim.x) a.key[base + i] = S.key[i];
    return 1;
}

}  // namespace
