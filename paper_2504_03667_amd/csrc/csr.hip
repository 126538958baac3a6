// Graphs stored as adjacency lists (CSR): the paper's sparse family (m = 3n
// edges, Section IV-A) without the n x n matrix whose memory the paper names as
// a weakness (the third point of Section V, the conclusion).  G[u][v] is the
// smallest weight of the edges u -> v; self-loops and weights outside
// [0, INT32_MAX) play no part, exactly as for a matrix built from the same edge
// list.
//
// Such graphs have many distinct distances and few edges, so the solve uses the
// label-correcting method (the paper's CUDA design, Algorithms 3 and 4, made
// deterministic in its results) over edges:
//   * a persistent grid of the workgroups that are on the GPU when the launch
//     starts (close_team); sweep k relaxes the edge lists of the
//     vertices whose dist dropped in sweep k-1 (the first frontier is the
//     source) with an agent-scope atomic minimum on the head's running dist;
//     the first lowering of a vertex in a sweep appends it to the next
//     frontier (three frontier lists rotate, so a list is cleared one sweep
//     before it is filled again); a sweep reads each tail's current dist, so
//     the sweep count can vary from run to run, the distances cannot;
//   * every word shared between workgroups is read and written with
//     agent-scope atomics (coherent across XCDs), so the barrier between
//     sweeps needs no cache writeback or invalidate;
//   * once no dist changes, one pass over all edges sets pred[v] to the tail u
//     of smallest (dist[u], u) among tight edges u -> v, u != v: Algorithm 1's
//     pred unless a tight edge has weight 0.  When one does, the order in
//     which Algorithm 1 settles equal distances decides pred, and a pass over
//     the vertices that tight zero-weight edges touch recovers that order
//     exactly (zero_tie_pred below), for any n.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <cstdarg>
#include <cstdio>

#include "engine.h"
#include "sssp.h"
#include "sssp_internal.h"

namespace sssp {
int set_error(int code, const char* msg);                                     // api.cpp
int stream_ctl(hipStream_t stream, Ctl** out, int* cus, long long* clock_khz);  // api.cpp
bool grid_launch_is_plain();                                                    // api.cpp
long long grid_barrier_ticks(long long clock_khz);                              // api.cpp
int served_workgroups(int device);                                              // server.cpp

namespace {

int err(int code, const char* fmt, ...) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    return set_error(code, buf);
}

constexpr int kCsrThreads = 1024;

// Control words of one CSR solve (device memory, zeroed by k_csr_init).
struct CsrCtl {
    uint32_t bar;  // barrier arrivals
    uint32_t pad0[31];
    uint64_t gen;  // (last completed barrier << 32) | the value it hands over
    uint32_t pad1[30];
    uint32_t count[3];    // frontier list sizes of the distance sweeps
    uint32_t zero;        // a tight zero-weight edge was seen
    uint32_t neg;         // a negative weight was seen
    uint32_t nlev;        // zero_tie_pred: levels holding non-plain vertices
    uint32_t next_level;  // zero_tie_pred: levels claimed by workgroups
    uint32_t solo_f, solo_tag;  // frontier and sweep number that workgroup 0 hands over (frontier_sweeps)
    uint32_t rest[3];     // smallest dist beyond the threshold, by scan number mod 3
    uint32_t delta;       // distances handled at a time (kInf: all)
    uint32_t pad2[18];
    uint32_t join;  // workgroups that have arrived; kTeamClosed: no more are taken
    uint32_t pad3[31];
    uint64_t team;  // (workgroups of the team << 32) | the first frontier it is handed; 0 before that
    uint32_t pad4[30];
};

// Scratch of zero_tie_pred (device memory; n = vertices, H = 2^hbits >= 2n).
struct ZeroTie {
    uint32_t* flags;   // per vertex: kNonPlain | kSeed | kAvail | kDone
    uint32_t* lev;     // per non-plain vertex: the number of its level
    uint32_t* seg;     // the non-plain vertices, grouped by level
    uint32_t* cnt;     // per level: its non-plain vertices
    uint32_t* off;     // per level: where its group starts in seg
    uint32_t* fill;    // per level: vertices placed in its group so far
    uint32_t* md;      // per vertex: smallest dist of a tail of a tight edge into it
    uint64_t* ht_key;  // open-addressing table of the levels' distances (H entries)
    uint32_t* ht_lvl;  // level number of each occupied table entry
    uint32_t hbits;
};

__device__ __forceinline__ bool edge_ok(int32_t u, int32_t v, int32_t w, int32_t n) {
    return v >= 0 && v < n && v != u && w >= 0 && w != (int32_t)kInf;
}

// ---------------------------------------------------------------------------
// Edge list -> CSR.
// ---------------------------------------------------------------------------

// Edges kept: endpoints in [0, n), weight in [0, INT32_MAX), not a self-loop.
__device__ __forceinline__ bool keep_edge(int32_t u, int32_t v, int32_t w, int32_t n) {
    return u >= 0 && u < n && v >= 0 && v < n && u != v && w >= 0 && w != (int32_t)kInf;
}

// Scratch of an edge list conversion (device memory).
struct ConvertScratch {
    unsigned long long* out;  // [0] edges left out, [1] entries of the lists
    uint32_t* deg;            // per vertex: entries of its list
    uint32_t* rank;           // per edge (undirected: then again for its other end): its place in the tail's list
    uint32_t* cursor;         // per vertex: entries placed so far; only where rank is null
    unsigned long long* sums; // per chunk of vertices: its entries
};

// Counts the lists' entries.  The count that an edge finds is its place in the
// tail's list, kept for k_csr_fill: bound by the atomics, which are then done once
// instead of again over cursors (see sssp_edges_to_csr for the figures).
__global__ void k_csr_degree(const int32_t* __restrict__ eu, const int32_t* __restrict__ ev,
                             const int32_t* __restrict__ ew, int64_t m, int32_t n, int32_t directed,
                             ConvertScratch cs) {
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < m; e += (int64_t)gridDim.x * blockDim.x) {
        const int32_t u = eu[e], v = ev[e], w = ew[e];
        const bool self = u == v && u >= 0 && u < n && w >= 0 && w != (int32_t)kInf;
        if (!keep_edge(u, v, w, n)) {
            if (!self) atomicAdd(&cs.out[0], 1ull);  // a valid self-loop is ignored, not an error
            continue;
        }
        const uint32_t ru = atomicAdd(&cs.deg[u], 1u);
        const uint32_t rv = directed ? 0u : atomicAdd(&cs.deg[v], 1u);
        if (cs.rank) {
            cs.rank[e] = ru;
            if (!directed) cs.rank[m + e] = rv;
        }
    }
}

// row_ptr[0] = 0, row_ptr[i + 1] = row_ptr[i] + deg[i], in passes over chunks of
// 1024 vertices: each chunk's total, then each chunk's scan plus its offset, the
// sum of the totals before it.  With more than kScanDirect chunks one workgroup
// scans the totals in between (each workgroup would read them all otherwise).
constexpr int kScanChunk = 1024;
constexpr int kScanDirect = 4096;

// Inclusive scan of one value per thread over a workgroup of kScanChunk
// threads; *total gets the workgroup's sum.
__device__ __forceinline__ unsigned long long wg_inclusive_scan(unsigned long long x, unsigned long long* wsum,
                                                                unsigned long long* total) {
    const int lane = threadIdx.x & 63;
    for (int o = 1; o < 64; o <<= 1) {
        const unsigned long long y = __shfl_up(x, (unsigned)o, 64);
        if (lane >= o) x += y;
    }
    if (lane == 63) wsum[threadIdx.x >> 6] = x;
    __syncthreads();
    unsigned long long before = 0, sum = 0;
    for (int k = 0; k < kScanChunk / 64; ++k) {
        if (k < (int)(threadIdx.x >> 6)) before += wsum[k];
        sum += wsum[k];
    }
    __syncthreads();  // wsum is reused by the next call
    *total = sum;
    return before + x;
}

__global__ __launch_bounds__(kScanChunk) void k_csr_chunk_sums(const uint32_t* __restrict__ deg, int32_t n,
                                                               unsigned long long* __restrict__ sums) {
    __shared__ unsigned long long wsum[kScanChunk / 64];
    const int64_t i = (int64_t)blockIdx.x * kScanChunk + threadIdx.x;
    unsigned long long total = 0;
    (void)wg_inclusive_scan(i < n ? deg[i] : 0ull, wsum, &total);
    if (threadIdx.x == 0) sums[blockIdx.x] = total;
}

// Exclusive scan of the chunk totals in place.
__global__ __launch_bounds__(kScanChunk) void k_csr_scan_sums(unsigned long long* __restrict__ sums, int32_t chunks) {
    __shared__ unsigned long long wsum[kScanChunk / 64];
    unsigned long long carry = 0;
    for (int32_t base = 0; base < chunks; base += kScanChunk) {
        const int32_t i = base + (int32_t)threadIdx.x;
        const unsigned long long x = i < chunks ? sums[i] : 0ull;
        unsigned long long total = 0;
        const unsigned long long incl = wg_inclusive_scan(x, wsum, &total);
        if (i < chunks) sums[i] = carry + incl - x;
        carry += total;
    }
}

// direct: sums holds the totals, else their exclusive scan.  *entries = row_ptr[n].
__global__ __launch_bounds__(kScanChunk) void k_csr_scan_chunks(const uint32_t* __restrict__ deg, int32_t n,
                                                                const unsigned long long* __restrict__ sums,
                                                                bool direct, int64_t* __restrict__ row_ptr,
                                                                unsigned long long* __restrict__ entries) {
    __shared__ unsigned long long wsum[kScanChunk / 64];
    unsigned long long total = 0, before = 0;
    if (direct) {
        unsigned long long x = 0;
        for (uint32_t k = threadIdx.x; k < blockIdx.x; k += kScanChunk) x += sums[k];
        (void)wg_inclusive_scan(x, wsum, &before);
    } else {
        before = sums[blockIdx.x];
    }
    const int64_t i = (int64_t)blockIdx.x * kScanChunk + threadIdx.x;
    const unsigned long long incl = wg_inclusive_scan(i < n ? deg[i] : 0ull, wsum, &total);
    if (i < n) row_ptr[i + 1] = (int64_t)(before + incl);
    if (i == 0) row_ptr[0] = 0;
    if (i == n - 1) *entries = before + incl;
}

__global__ void k_csr_fill(const int32_t* __restrict__ eu, const int32_t* __restrict__ ev,
                           const int32_t* __restrict__ ew, int64_t m, int32_t n, int32_t directed,
                           const int64_t* __restrict__ row_ptr, ConvertScratch cs, int32_t* __restrict__ col,
                           int32_t* __restrict__ w) {
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < m; e += (int64_t)gridDim.x * blockDim.x) {
        const int32_t u = eu[e], v = ev[e], wt = ew[e];
        if (!keep_edge(u, v, wt, n)) continue;
        int64_t p = row_ptr[u] + (cs.rank ? cs.rank[e] : atomicAdd(&cs.cursor[u], 1u));
        col[p] = v;
        w[p] = wt;
        if (!directed) {
            p = row_ptr[v] + (cs.rank ? cs.rank[m + e] : atomicAdd(&cs.cursor[v], 1u));
            col[p] = u;
            w[p] = wt;
        }
    }
}

__device__ __forceinline__ uint64_t entry_key(int32_t v, int32_t w) {  // both >= 0: compares as (head, weight)
    return (uint64_t)(uint32_t)v << 32 | (uint32_t)w;
}

// Sorts col[0, len), w[0, len) by (head, weight); all lanes of a wave call it.
// Bitonic merges whose every exchange puts the smaller entry first, so entries
// beyond len, thought of as largest, never move and need not exist.
__device__ void sort_long_row(int32_t* col, int32_t* w, int64_t len) {
    for (int64_t k = 2; k < 2 * len; k <<= 1) {
        for (int64_t j = k >> 1; j > 0; j >>= 1) {
            const bool flip = j == k >> 1;  // the first exchange of a merge mirrors its second half
            for (int64_t p = wave_lane(); p < len; p += kWave) {
                const int64_t in = p & (j - 1), lo = 2 * (p - in) + in;
                const int64_t hi = flip ? lo + 2 * (j - in) - 1 : lo + j;
                if (hi >= len) continue;
                const int32_t cl = col[lo], ch = col[hi], wl = w[lo], wh = w[hi];
                if (entry_key(cl, wl) > entry_key(ch, wh)) {
                    col[lo] = ch;
                    col[hi] = cl;
                    w[lo] = wh;
                    w[hi] = wl;
                }
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");  // the wave's stores before its next loads
            __builtin_amdgcn_wave_barrier();
        }
    }
}

// Sort each row by (head, weight) so that the lists do not depend on the order
// the atomics above took.  A wave takes eight rows: eight lanes count for each
// entry of a row of up to 8 how many precede it and store it there, rows of up to
// 64 are taken the same way by the whole wave one after the other, longer ones are
// sorted in place.  Bound by the latency of one load and one store a row, where a
// thread a row moved entries one by one through memory (see sssp_edges_to_csr).
__global__ __launch_bounds__(256) void k_csr_sort_rows(const int64_t* __restrict__ row_ptr, int32_t n, int32_t* col,
                                                       int32_t* w) {
    constexpr int kLanes = 8;
    const int lane = wave_lane();
    const int sub = lane % kLanes;
    const int64_t wave = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / kWave;
    const int64_t waves = (int64_t)gridDim.x * blockDim.x / kWave;
    for (int64_t u0 = wave * (kWave / kLanes); u0 < n; u0 += waves * (kWave / kLanes)) {
        const int64_t u = u0 + lane / kLanes;
        int64_t a = 0, len = 0;
        if (u < n) {
            a = row_ptr[u];
            len = row_ptr[u + 1] - a;
        }
        const bool mine = len <= kLanes && sub < len;
        int32_t c = 0, x = 0;
        if (mine) {
            c = col[a + sub];
            x = w[a + sub];
        }
        uint32_t pos = 0;
#pragma unroll
        for (int j = 0; j < kLanes; ++j) {
            const uint64_t other = entry_key(__shfl(c, j, kLanes), __shfl(x, j, kLanes));
            const uint64_t key = entry_key(c, x);
            pos += j < len && (other < key || (other == key && j < sub)) ? 1u : 0u;
        }
        if (mine) {
            col[a + pos] = c;
            w[a + pos] = x;
        }
        for (uint64_t rest = __ballot(sub == 0 && len > kLanes); rest; rest &= rest - 1) {
            const int64_t v = u0 + (__ffsll((unsigned long long)rest) - 1) / kLanes;
            const int64_t av = row_ptr[v], lv = row_ptr[v + 1] - av;
            if (lv > kWave) {
                sort_long_row(col + av, w + av, lv);
                continue;
            }
            c = x = 0;
            if (lane < lv) {
                c = col[av + lane];
                x = w[av + lane];
            }
            const uint64_t key = entry_key(c, x);
            pos = 0;
            for (int j = 0; j < (int)lv; ++j) {
                const uint64_t other = entry_key(__builtin_amdgcn_readlane(c, j), __builtin_amdgcn_readlane(x, j));
                pos += other < key || (other == key && j < lane) ? 1u : 0u;
            }
            if (lane < lv) {
                col[av + pos] = c;
                w[av + pos] = x;
            }
        }
    }
}

// ---------------------------------------------------------------------------
// Solve.
//
// Labels: a running value (dist) and the sweep that last
// lowered it, packed as (value << 32) | sweep into one 64-bit word.  Sweep
// numbers grow, so an atomic minimum with (c << 32) | k lowers the value
// exactly when c is smaller (a tie keeps the older word), and the word it
// returns tells whether sweep k had already lowered it: only the first
// lowering of a vertex in a sweep appends it to the next frontier.
// ---------------------------------------------------------------------------

__device__ __forceinline__ uint32_t label_value(uint64_t x) { return (uint32_t)(x >> 32); }

// Graphs from which the sweeps take a range of distances at a time (see
// frontier_sweeps), if their lists hold four entries a vertex on average (graphs of
// long chains gain nothing).  Below, sweeps are bound by latency and the extra ones
// cost more than the relaxations they save.  Undirected, m=3n, sweeps and lists
// relaxed without and with ranges: n=40000 23 and 121 thousand against 29 and 50
// (302 us and 320), n=100000 26 and 363 against 38 and 140 (394 and 405), n=200000
// 27 and 724 against 39 and 283 (518 and 494), n=10^6 32 and 3.7 million against 45
// and 1.3 (2.5 ms and 1.1).
constexpr int32_t kRangeMinN = 131072;
constexpr int kWeightSample = 256;
// A range of distances is this many times the mean weight over the mean list
// length, so that a vertex has about as many edges within a range at any density
// (8 to 18 tried: n=10^6 of 6 a vertex 1197, 1087, 1372 us at 8, 12, 18; of 20 a
// vertex 2420, 2235, 2982; twice the mean weight at any density 1.1 and 4.25 ms).
constexpr double kRangeEdges = 12;

__global__ void k_csr_init(int32_t n, int32_t src, const int64_t* __restrict__ row_ptr, const int32_t* __restrict__ w,
                           uint64_t* __restrict__ lab, uint64_t* __restrict__ pkey, uint32_t* __restrict__ lists,
                           CsrCtl* __restrict__ cc) {
    if (blockIdx.x == 0 && n >= kRangeMinN) {
        // the range, from the mean weight of a sample spread over the lists
        __shared__ unsigned long long sum;
        __shared__ uint32_t count;
        if (threadIdx.x == 0) {
            sum = 0;
            count = 0;
        }
        __syncthreads();
        const int64_t m = row_ptr[n];
        for (int i = threadIdx.x; i < kWeightSample && m > 0; i += blockDim.x) {
            const int32_t x = w[(int64_t)i * m / kWeightSample];
            if (x >= 0 && x != (int32_t)kInf) {
                atomicAdd(&sum, (unsigned long long)x);
                atomicAdd(&count, 1u);
            }
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            const double d = count && m >= 4 * (int64_t)n ? kRangeEdges * (double)n * (double)sum / ((double)m * count) : 0;
            cc->delta = d < 1 || d >= (double)kInf ? kInf : (uint32_t)d;
        }
    }
    const int64_t gtid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    for (int64_t v = gtid; v < n; v += (int64_t)gridDim.x * blockDim.x) {
        lab[v] = v == src ? 0ull : (uint64_t)kInf << 32;
        pkey[v] = kNoKey;
    }
    if (gtid == 0) {
        lists[0] = (uint32_t)src;
        cc->bar = 0;
        cc->gen = 0ull;
        for (int i = 0; i < 3; ++i) cc->count[i] = i == 0 ? 1u : 0u;
        cc->zero = 0;
        cc->neg = 0;
        cc->nlev = 0;
        cc->next_level = 0;
        for (int i = 0; i < 3; ++i) cc->rest[i] = kInf;
        cc->join = 0;
        cc->team = 0;
        if (n < kRangeMinN) cc->delta = kInf;
    }
}

// Grid barrier b of nwg workgroups.  Everything shared goes through agent-scope
// atomics, whose completion each wave waits for before the workgroup barrier,
// so an arrival counter and a release word suffice.  The last workgroup to
// arrive reads *carry (when given: by then every other workgroup's atomics on
// it have completed) and hands it to all in the release word, saving each
// workgroup that read.  false: a wait gave up.
__device__ __forceinline__ bool csr_barrier(CsrCtl* cc, uint32_t b, uint32_t nwg, long long timeout,
                                            const uint32_t* carry = nullptr, uint32_t* value = nullptr) {
    __shared__ uint32_t handed;
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    int late = 0;
    if (threadIdx.x == 0) {
        uint32_t val = 0;
        if (nwg == 1) {
            if (carry) val = ld_agent(carry);
        } else {
            stress_delay(b);
            const uint32_t old = __hip_atomic_fetch_add(&cc->bar, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (old == b * nwg - 1) {
                if (carry) val = ld_agent(carry);
                st_agent(&cc->gen, ((uint64_t)b << 32) | val);
            } else {
                const long long t0 = wall_clock64();
                unsigned naps = 1;
                uint64_t g = ld_agent(&cc->gen);
                while ((uint32_t)(g >> 32) < b) {
                    for (unsigned i = 0; i < naps; ++i) __builtin_amdgcn_s_sleep(1);
                    if (naps < 8) naps <<= 1;
                    if (wall_clock64() - t0 > timeout) {
                        late = 1;
                        break;
                    }
                    g = ld_agent(&cc->gen);
                }
                val = (uint32_t)g;
            }
        }
        handed = val;
    }
    const bool ok = __syncthreads_or(late) == 0;
    if (value) *value = handed;
    return ok;
}

// The workgroups that take part.  A grid barrier waits for all of its workgroups, and
// other work can keep some from starting for as long as it runs (a resident server
// holds nearly every compute unit), so the grid's size is what is asked for and the
// team's is what has come: each workgroup's arrival gives it its rank, and the first,
// once it has done what it does alone, waits up to `limit` ticks for the rest, then
// closes the team and hands it the frontier.  Later ones find it closed and leave.
// close_team is the team's first barrier; false: the first workgroup's word did not
// come within `timeout`.
constexpr uint32_t kTeamClosed = 0x80000000u;
// Waiting longer than a solve takes is no gain: the smallest wait that covers the start
// of a grid on an idle GPU many times over.
constexpr int kTeamWaitUs = 200;

__device__ __forceinline__ uint32_t join_team(CsrCtl* cc) {
    __shared__ uint32_t rank;
    if (threadIdx.x == 0) {
        stress_delay(0x7ea3u);
        rank = __hip_atomic_fetch_add(&cc->join, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    return scalar(rank);
}

__device__ __forceinline__ bool close_team(CsrCtl* cc, uint32_t rank, uint32_t asked, long long limit,
                                           long long timeout, uint32_t& size, uint32_t& F) {
    __shared__ uint64_t handed;
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if (threadIdx.x == 0) {
        const long long t0 = wall_clock64();
        uint64_t team = 0;
        if (rank == 0) {
            uint32_t k = ld_agent(&cc->join);
            while (k < asked && wall_clock64() - t0 < limit) {
                __builtin_amdgcn_s_sleep(1);
                k = ld_agent(&cc->join);
            }
            k = __hip_atomic_fetch_or(&cc->join, kTeamClosed, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            team = ((uint64_t)k << 32) | F;
            st_agent(&cc->team, team);
        } else {
            unsigned naps = 1;
            while ((team = ld_agent(&cc->team)) == 0 && wall_clock64() - t0 <= timeout) {
                for (unsigned i = 0; i < naps; ++i) __builtin_amdgcn_s_sleep(1);
                if (naps < 8) naps <<= 1;
            }
        }
        handed = team;
    }
    __syncthreads();
    size = scalar((uint32_t)(handed >> 32));
    F = scalar((uint32_t)handed);
    return size != 0;
}

// Number of this wave in the team, neighbours in different workgroups: long lists of
// vertices whose indices are close, in the passes over all of them, and a frontier handed
// back for its long lists are then spread over the compute units.  (Other sweeps take
// neighbours in one workgroup, as they have their heads in common and few workgroups'
// appends to gather: a torus of 10^6 vertices 6.4 ms against 7.8.)
__device__ __forceinline__ int64_t team_wave(uint32_t rank, uint32_t nwg) {
    return (int64_t)(threadIdx.x / kWave) * nwg + rank;
}
__device__ __forceinline__ int64_t team_thread(uint32_t rank, uint32_t nwg) {
    return team_wave(rank, nwg) * kWave + (threadIdx.x & (kWave - 1));
}

// Does tail u (dist du) reach head v (dist dv) over an edge of weight wt on a
// shortest path?  Both finite, du + wt == dv (both below 2^31: no wrap).
__device__ __forceinline__ bool tight(uint32_t du, uint32_t dv, int32_t wt) {
    return du < kInf && dv < kInf && du + (uint32_t)wt == dv;
}

// Frontier sweeps over three rotating lists whose sizes are count[0..2]; the
// first frontier (F vertices) is in list 0.  A group of G lanes takes one
// frontier vertex u and walks its edge list G * B edges per step, every load
// and atomic of a step in flight together: value(tail(u), u, v, w, c) says
// whether edge u -> v takes part and gives its candidate c, and an atomic
// minimum of (c << 32) | sweep on lab[v] lowers v; its first lowering below the
// threshold in the sweep appends v to the next frontier.  Appends are gathered in
// LDS and take one counter update per workgroup and sweep: one per wave and step
// is thousands of updates of one word a sweep at n=10^6.
// A list therefore holds a vertex at most once; the list read in one sweep is
// cleared in the next and filled in the one after.  Medium frontiers are bound
// by latency: 16 lanes share a vertex, so that most lists take one step and more
// waves have work (n=40000, m=16n: 4 lanes of 2 edges 803 us, 8 lanes 645, 16 lanes
// 575).  Large ones are bound by memory operations: each head is read first and the
// atomic skipped when the edge cannot lower it (8 lanes of 2 edges; a lane a list,
// 8 edges a step: n=10^6 1094 us against 966).  Small ones (half of the sweeps or
// more) are left to workgroup 0, which keeps them in LDS and needs no grid barrier
// between them; the others wait at the barrier that ends its run.  Where lists are
// long on average one workgroup would take longer over them than the barriers take, and
// a vertex of a long list it leaves to all: it joins the frontier that is handed back
// (400 lists of 5000 entries reached at once: 2.7 ms, with workgroup 0 alone 12.3).
// Large graphs take a range of distances at a time: vertices lowered to thr or
// above are not relaxed yet, and when the frontier is empty a scan of the labels
// gathers those of the next range (nothing below the old threshold is left to
// relax, and nothing above it has been), which saves most repeated relaxations.
// Solves of m=3n before (no ranges, one append a wave and step, a barrier a sweep)
// and now: n=1000 133 -> 115 us, 10000 207 -> 174, 40000 368 -> 248, 200000 824 ->
// 390, 10^6 2670 -> 980 (event to event, scratch allocation included).
constexpr uint32_t kLargeFrontier = 32768;
constexpr uint32_t kRangeFew = 256;  // vertices of a range below which the next ones are twice as wide: the sample
                                     // misjudges a graph whose paths are not made of its typical edges
constexpr uint32_t kSoloFrontier = 512;  // n=10000: 256 209 us, 512 212, 768 215, 1536 253
constexpr int64_t kSoloDegree = 16;     // only if the lists are this short on average
constexpr int64_t kSoloList = 64;       // ... and of a vertex that workgroup 0 relaxes: longer lists it hands back
constexpr uint32_t kWide = 0x80000000u;  // mark of a frontier handed back for that (the next sweep is everybody's)
constexpr uint32_t kAppendCap = 4096;   // entries gathered in LDS

struct SweepLds {
    uint32_t buf[kAppendCap];
    uint32_t longs[kSoloFrontier];
    uint32_t nlong[2];
    uint32_t fill[2];
    uint32_t base;
    uint32_t rest;
};

// The wave's appends: `want` marks v[j] of the lane.  Positions come from *fill;
// entries that do not fit `room` go to `over`: at positions that one update of the
// counter over_count takes for the wave, or at the ones found if that is null.  (With
// an update for each entry n=1.2*10^7, m=6n, where a workgroup's sweep appends far more
// than fits, took 15 to 55 ms by source, with one a wave 13 to 35.)
template <int B>
__device__ __forceinline__ void append(uint32_t want, const int32_t (&v)[B], uint32_t* buf, uint32_t room,
                                       uint32_t* fill, uint32_t* __restrict__ over, uint32_t* __restrict__ over_count) {
    const uint32_t mine = (uint32_t)__popc(want);
    const uint32_t incl = wave_prefix32(mine);
    const uint32_t total = lane_value(incl, kWave - 1);
    if (!total) return;
    uint32_t at = 0;
    if (wave_lane() == 0)
        at = __hip_atomic_fetch_add(fill, total, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    at = lane_value(at, 0);
    uint32_t pos = at + incl - mine;
    uint32_t shift = 0;  // from a position beyond the room to the one in `over`
    if (over_count && at + total > room) {
        const uint32_t first = max(at, room);
        uint32_t q = 0;
        if (wave_lane() == 0)
            q = __hip_atomic_fetch_add(over_count, at + total - first, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        shift = lane_value(q, 0) - first;
    }
#pragma unroll
    for (int j = 0; j < B; ++j)
        if (want >> j & 1u) {
            if (pos < room) buf[pos] = (uint32_t)v[j];
            else st_agent(&over[pos + shift], (uint32_t)v[j]);
            ++pos;
        }
}

// One sweep over frontier entries entry(i), i < F, by the waves wave, wave + waves, ...
// With `longs`, vertices whose lists are longer than kSoloList are put there (*nlong
// counts them) and not relaxed.
template <int G, int B, bool Filter, class Entry, class Tail, class Value>
__device__ __forceinline__ void sweep_frontier(Entry entry, uint32_t F, int64_t wave, int64_t waves, uint32_t* buf,
                                               uint32_t room, uint32_t* fill, uint32_t* __restrict__ over,
                                               uint32_t* __restrict__ over_count, uint64_t* __restrict__ lab,
                                               const int64_t* __restrict__ row_ptr, const int32_t* __restrict__ col,
                                               const int32_t* __restrict__ w, uint32_t tag, uint32_t thr, Tail& tail,
                                               Value& value, uint32_t* longs = nullptr, uint32_t* nlong = nullptr) {
    const int lane = threadIdx.x & (kWave - 1);
    const int sub = lane % G;
    const int64_t per_wave = kWave / G;
    for (int64_t i0 = wave * per_wave; i0 < (int64_t)F; i0 += waves * per_wave) {  // the same trip count in a wave
        const int64_t i = i0 + lane / G;
        int32_t u = 0;
        decltype(tail(0)) tv{};
        int64_t e = 0, e1 = 0;
        if (i < (int64_t)F) {
            u = (int32_t)entry((uint32_t)i);
            tv = tail(u);
            e = row_ptr[u] + sub;
            e1 = row_ptr[u + 1];
            if (longs && e1 - e > kSoloList - sub) {
                if (sub == 0)
                    longs[__hip_atomic_fetch_add(nlong, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)] = (uint32_t)u;
                e = e1;
            }
        }
        while (__ballot(e < e1)) {
            int32_t v[B];
            uint32_t c[B];
            uint64_t before[B];
            bool part[B];
#pragma unroll
            for (int j = 0; j < B; ++j) {
                const int64_t ej = e + (int64_t)j * G;
                part[j] = false;
                v[j] = 0;
                c[j] = 0;
                if (ej < e1) {
                    v[j] = col[ej];
                    part[j] = value(tv, u, v[j], w[ej], c[j]);
                }
            }
            if (Filter) {
                uint64_t now[B];
#pragma unroll
                for (int j = 0; j < B; ++j) now[j] = part[j] ? ld_agent(&lab[v[j]]) : 0ull;
#pragma unroll
                for (int j = 0; j < B; ++j) part[j] = part[j] && c[j] < label_value(now[j]);
            }
#pragma unroll
            for (int j = 0; j < B; ++j)
                before[j] = part[j] ? __hip_atomic_fetch_min(&lab[v[j]], ((uint64_t)c[j] << 32) | tag, __ATOMIC_RELAXED,
                                                             __HIP_MEMORY_SCOPE_AGENT)
                                    : 0ull;
            uint32_t want = 0;
#pragma unroll
            for (int j = 0; j < B; ++j)
                want |= (part[j] && c[j] < thr && c[j] < label_value(before[j]) &&
                                 ((uint32_t)before[j] != tag || label_value(before[j]) >= thr)
                             ? 1u : 0u) << j;
            append<B>(want, v, buf, room, fill, over, over_count);
            e += (int64_t)G * B;
        }
    }
}

// The workgroup's gathered appends to the next list (every thread calls it).
__device__ __forceinline__ void flush_appends(SweepLds& sl, uint32_t* __restrict__ next,
                                              uint32_t* __restrict__ next_count) {
    __syncthreads();
    const uint32_t k = min(sl.fill[0], kAppendCap);
    if (k) {
        if (threadIdx.x == 0)
            sl.base = __hip_atomic_fetch_add(next_count, k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __syncthreads();
        const uint32_t base = sl.base;
        for (uint32_t i = threadIdx.x; i < k; i += blockDim.x) st_agent(&next[base + i], sl.buf[i]);
    }
    __syncthreads();
    if (threadIdx.x == 0) sl.fill[0] = 0;
    // ordered before the next sweep's appends by the barrier that follows
}

// The barrier that ends a sweep hands over the next frontier's size.  Stops when
// no vertex is left to relax; false if a barrier wait gave up.  rank: this
// workgroup's; nwg gets the number of workgroups (close_team).
template <class Tail, class Value>
__device__ bool frontier_sweeps(uint32_t rank, uint32_t& nwg, long long team_limit,
                                uint32_t* __restrict__ count, uint32_t* __restrict__ lists,
                                uint64_t* __restrict__ lab, const int64_t* __restrict__ row_ptr,
                                const int32_t* __restrict__ col, const int32_t* __restrict__ w, int32_t n, CsrCtl* cc,
                                uint32_t& b, long long timeout, uint32_t F, unsigned long long& sweeps,
                                unsigned long long& rows, SweepLds& sl, Tail tail, Value value) {
    const int wgwaves = (int)(blockDim.x / kWave);
    const int64_t wave = (int64_t)rank * wgwaves + threadIdx.x / kWave;
    int64_t waves = 0;
    uint32_t delta = cc->delta;  // written by the launch before this one
    const uint32_t solo = row_ptr[n] <= kSoloDegree * n ? kSoloFrontier : 0u;
    uint32_t thr = delta, tag = 0, ph = 0, scans = 0;
    nwg = 0;
    if (threadIdx.x < 2) sl.fill[threadIdx.x] = sl.nlong[threadIdx.x] = 0;
    __syncthreads();
    bool wide = false;
    for (;;) {
        while (F) {
            if ((F <= solo && !wide) || nwg == 0) {
                if (rank == 0 && F <= solo) {
                    constexpr uint32_t half = kAppendCap / 2;
                    uint32_t* cur = sl.buf;
                    uint32_t* nxt = sl.buf + half;
                    for (uint32_t i = threadIdx.x; i < F; i += blockDim.x)
                        cur[i] = ld_agent(&lists[(size_t)ph * n + i]);
                    __syncthreads();
                    uint32_t k = 0, L = 0;
                    bool hand_back = false;
                    const long long t_solo = wall_clock64();
                    do {
                        ++sweeps;
                        rows += F;
                        ++tag;
                        uint32_t* fill = &sl.fill[k & 1];
                        sweep_frontier<4, 2, false>([&](uint32_t i) { return cur[i]; }, F, threadIdx.x / kWave, wgwaves,
                                                    nxt, half, fill, lists, nullptr, lab, row_ptr, col, w, tag, thr,
                                                    tail, value, sl.longs, &sl.nlong[k & 1]);
                        __syncthreads();
                        F = *fill;
                        L = sl.nlong[k & 1];
                        if (L && (uint64_t)F + L > (uint64_t)n) {
                            // no room in a list of n for vertices that may be in it twice
                            __syncthreads();
                            sweep_frontier<4, 2, false>([&](uint32_t i) { return sl.longs[i]; }, L,
                                                        threadIdx.x / kWave, wgwaves, nxt, half, fill, lists, nullptr,
                                                        lab, row_ptr, col, w, tag, thr, tail, value);
                            __syncthreads();
                            F = *fill;
                            L = 0;
                        }
                        if (threadIdx.x == 0) {
                            sl.fill[(k & 1) ^ 1] = sl.nlong[(k & 1) ^ 1] = 0;
                            // the waiting workgroups' limit must not be reached by a run of slow
                            // sweeps (vertices of very long lists) that each stay below it
                            sl.base = wall_clock64() - t_solo > timeout / 4 ? 1u : 0u;
                        }
                        uint32_t* t = cur;
                        cur = nxt;
                        nxt = t;
                        __syncthreads();
                        hand_back = sl.base != 0 || L != 0;
                        ++k;
                    } while (F && F <= solo && !hand_back);
                    // the frontier into list 0 (what did not fit LDS is there already)
                    for (uint32_t i = threadIdx.x; i < min(F, half); i += blockDim.x) st_agent(&lists[i], cur[i]);
                    for (uint32_t i = threadIdx.x; i < L; i += blockDim.x) st_agent(&lists[F + i], sl.longs[i]);
                    F = (F + L) | (L ? kWide : 0u);
                    __syncthreads();
                    if (threadIdx.x == 0) {
                        sl.fill[0] = sl.fill[1] = sl.nlong[0] = sl.nlong[1] = 0;
                        st_agent(&count[1], 0u);
                        st_agent(&count[2], 0u);
                        st_agent(&cc->solo_tag, tag);
                        st_agent(&cc->solo_f, F);
                    }
                }
                if (nwg == 0) {
                    if (!close_team(cc, rank, gridDim.x, team_limit, timeout, nwg, F)) return false;
                    waves = (int64_t)nwg * wgwaves;
                } else if (!csr_barrier(cc, ++b, nwg, timeout, &cc->solo_f, &F)) {
                    return false;
                }
                if (solo) tag = ld_agent(&cc->solo_tag);
                wide = (F & kWide) != 0;
                F &= ~kWide;
                ph = 0;
                continue;
            }
            const int64_t at = wide ? team_wave(rank, nwg) : wave;
            wide = false;
            const uint32_t nx = ph == 2 ? 0 : ph + 1, old = nx == 2 ? 0 : nx + 1;
            ++sweeps;
            rows += F;
            ++tag;
            if (rank == 0 && threadIdx.x == 0) st_agent(&count[old], 0u);
            const uint32_t* list = lists + (size_t)ph * n;
            uint32_t* next = lists + (size_t)nx * n;
            auto entry = [&](uint32_t i) { return ld_agent(&list[i]); };
            if (F >= kLargeFrontier)
                sweep_frontier<8, 2, true>(entry, F, wave, waves, sl.buf, kAppendCap, &sl.fill[0], next, &count[nx],
                                           lab, row_ptr, col, w, tag, thr, tail, value);
            else
                sweep_frontier<16, 1, false>(entry, F, at, waves, sl.buf, kAppendCap, &sl.fill[0], next, &count[nx],
                                            lab, row_ptr, col, w, tag, thr, tail, value);
            flush_appends(sl, next, &count[nx]);
            if (!csr_barrier(cc, ++b, nwg, timeout, &count[nx], &F)) return false;
            ph = nx;
        }
        if (thr >= kInf) return true;
        // the next range: open labels from thr on, and the smallest beyond it
        const uint32_t nx = ph == 2 ? 0 : ph + 1, old = nx == 2 ? 0 : nx + 1;
        const uint32_t end = (uint32_t)min((uint64_t)thr + delta, (uint64_t)kInf);
        const uint32_t rs = scans % 3;
        if (rank == 0 && threadIdx.x == 0) {
            st_agent(&count[old], 0u);
            st_agent(&cc->rest[(scans + 1) % 3], kInf);
        }
        if (threadIdx.x == 0) sl.rest = kInf;
        __syncthreads();
        uint32_t* next = lists + (size_t)nx * n;
        uint32_t rest = kInf;
        for (int64_t v0 = wave * kWave; v0 < n; v0 += waves * kWave) {
            const int64_t v = v0 + (threadIdx.x & (kWave - 1));
            const uint32_t d = v < n ? label_value(ld_agent(&lab[v])) : kInf;
            if (d >= end) rest = min(rest, d);
            const int32_t vv[1] = {(int32_t)v};
            append<1>(d >= thr && d < end ? 1u : 0u, vv, sl.buf, kAppendCap, &sl.fill[0], next, &count[nx]);
        }
        rest = wave_min32(rest);
        if ((threadIdx.x & (kWave - 1)) == 0 && rest < kInf)
            __hip_atomic_fetch_min(&sl.rest, rest, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        flush_appends(sl, next, &count[nx]);
        if (threadIdx.x == 0 && sl.rest < kInf)
            __hip_atomic_fetch_min(&cc->rest[rs], sl.rest, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (!csr_barrier(cc, ++b, nwg, timeout, &count[nx], &F)) return false;
        ph = nx;
        ++scans;
        if (F < kRangeFew) delta = (uint32_t)min(2 * (uint64_t)delta, (uint64_t)kInf);
        if (F) {
            thr = end;
        } else {
            thr = ld_agent(&cc->rest[rs]);  // empty range: go on from the nearest vertex
            if (thr >= kInf) return true;
        }
    }
}

// Calls f(v[], w[], ok[]) for the edges of u, kBatch at a time, after loading
// them together; ok marks the edges that take part (edge_ok).
constexpr int kBatch = 4;
template <class F>
__device__ __forceinline__ void for_edges(const int64_t* __restrict__ row_ptr, const int32_t* __restrict__ col,
                                          const int32_t* __restrict__ w, int32_t n, int32_t u, F f) {
    const int64_t e1 = row_ptr[u + 1];
    for (int64_t e = row_ptr[u]; e < e1; e += kBatch) {
        int32_t v[kBatch], wt[kBatch];
        bool ok[kBatch];
#pragma unroll
        for (int j = 0; j < kBatch; ++j) {
            v[j] = 0;
            wt[j] = -1;
            if (e + j < e1) {
                v[j] = col[e + j];
                wt[j] = w[e + j];
            }
            ok[j] = e + j < e1 && edge_ok(u, v[j], wt[j], n);
        }
        f(v, wt, ok);
    }
}

// pred when tight zero-weight edges exist, from the exact distances alone
// (every workgroup of the grid calls it; b counts the grid barriers).
//
// Algorithm 1 settles vertices in order of distance, and within one distance
// (a level) it settles the lowest-index vertex whose dist already equals that
// distance: the seeds (the source, and heads of tight edges of positive weight,
// whose tails lie in lower levels) from the start, and the heads of tight
// zero-weight edges once their tail has settled.  pred[v] is the tail of the
// tight edge into v that settled first.  Vertices touched by no tight
// zero-weight edge inside their level ("plain") are seeds that make nothing
// available, so only the others ("non-plain") need a sequential pass, one
// level per workgroup: it settles them one at a time as Algorithm 1 would,
// y_1, y_2, ..., and a plain vertex p settles before y_i exactly when
// p < max(y_1 .. y_i).  Hence within a level the settle order is the order of
// the 64-bit keys p << 32 for plain p and (max(y_1 .. y_i) << 32) | i for y_i,
// and pred[v] is the tail u of smallest (dist[u], key[u]) over tight edges
// u -> v, u != v: found by a minimum of dist[u], then of key[u] among those
// tails, then the tail whose key won.  The non-plain vertices are grouped by
// level through an open-addressing table of the levels' distances.
constexpr uint32_t kNonPlain = 1u, kSeed = 2u, kAvail = 4u, kDone = 8u;
constexpr uint64_t kEmpty = ~0ull;

__device__ __forceinline__ uint32_t level_slot(uint32_t d, uint32_t hbits) {
    return (d * 2654435761u) >> (32 - hbits);
}

template <int T>
__device__ bool zero_tie_pred(uint32_t rank, uint32_t nwg, const int64_t* __restrict__ row_ptr,
                              const int32_t* __restrict__ col, const int32_t* __restrict__ w, int32_t n, int32_t src, const uint64_t* __restrict__ lab,
                              uint64_t* __restrict__ rk, uint64_t* __restrict__ pk, const ZeroTie& zt, CsrCtl* cc,
                              uint32_t& b, long long timeout, int32_t* __restrict__ dist,
                              int32_t* __restrict__ pred, Red<T>& red) {
    __shared__ uint32_t claim;
    const int64_t gtid = team_thread(rank, nwg);
    const int64_t gsz = (int64_t)nwg * T;
    const uint32_t hmask = (uint32_t)((1ull << zt.hbits) - 1ull);
    auto D = [&](int64_t v) { return label_value(ld_agent(&lab[v])); };
    auto set_flag = [&](int64_t v, uint32_t f) {
        __hip_atomic_fetch_or(&zt.flags[v], f, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    // every vertex starts plain with its own index as settle key; the table starts empty
    for (int64_t v = gtid; v < n; v += gsz) {
        st_agent(&zt.flags[v], v == src ? kSeed : 0u);
        st_agent(&zt.cnt[v], 0u);
        st_agent(&zt.fill[v], 0u);
        st_agent(&zt.md[v], kInf);
        st_agent(&rk[v], (uint64_t)v << 32);
        st_agent(&pk[v], kNoKey);
    }
    for (int64_t h = gtid; h <= (int64_t)hmask; h += gsz) st_agent(&zt.ht_key[h], kEmpty);
    if (!csr_barrier(cc, ++b, nwg, timeout)) return false;
    // tight zero-weight edges make both ends non-plain; positive ones make the head a seed
    for (int64_t u = gtid; u < n; u += gsz) {
        const uint32_t du = D(u);
        if (du >= kInf) continue;
        for_edges(row_ptr, col, w, n, (int32_t)u, [&](const int32_t* v, const int32_t* wt, const bool* eok) {
            uint32_t dv[kBatch];
#pragma unroll
            for (int j = 0; j < kBatch; ++j) dv[j] = eok[j] ? D(v[j]) : kInf;
#pragma unroll
            for (int j = 0; j < kBatch; ++j) {
                if (!tight(du, dv[j], wt[j])) continue;
                if (wt[j] == 0) {
                    set_flag(u, kNonPlain);
                    set_flag(v[j], kNonPlain);
                } else {
                    set_flag(v[j], kSeed);
                }
            }
        });
    }
    if (!csr_barrier(cc, ++b, nwg, timeout)) return false;
    // the distance of every non-plain vertex enters the table (one entry per level)
    for (int64_t v = gtid; v < n; v += gsz) {
        if (!(ld_agent(&zt.flags[v]) & kNonPlain)) continue;
        const uint64_t d = D(v);
        for (uint32_t h = level_slot((uint32_t)d, zt.hbits);; h = (h + 1) & hmask) {
            uint64_t expect = kEmpty;
            if (__hip_atomic_compare_exchange_strong(&zt.ht_key[h], &expect, d, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                     __HIP_MEMORY_SCOPE_AGENT) ||
                expect == d)
                break;
        }
    }
    if (!csr_barrier(cc, ++b, nwg, timeout)) return false;
    // number the levels
    for (int64_t h = gtid; h <= (int64_t)hmask; h += gsz)
        if (ld_agent(&zt.ht_key[h]) != kEmpty)
            st_agent(&zt.ht_lvl[h], __hip_atomic_fetch_add(&cc->nlev, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
    if (!csr_barrier(cc, ++b, nwg, timeout)) return false;
    // each non-plain vertex finds its level and counts itself in
    for (int64_t v = gtid; v < n; v += gsz) {
        if (!(ld_agent(&zt.flags[v]) & kNonPlain)) continue;
        const uint64_t d = D(v);
        uint32_t h = level_slot((uint32_t)d, zt.hbits);
        while (ld_agent(&zt.ht_key[h]) != d) h = (h + 1) & hmask;
        const uint32_t L = ld_agent(&zt.ht_lvl[h]);
        st_agent(&zt.lev[v], L);
        __hip_atomic_fetch_add(&zt.cnt[L], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (!csr_barrier(cc, ++b, nwg, timeout)) return false;
    const uint32_t nl = ld_agent(&cc->nlev);
    // where each level's group starts: an exclusive scan of the counts, by workgroup 0
    if (rank == 0) {
        uint32_t run = 0;
        for (uint32_t base = 0; base < nl; base += T) {
            const uint32_t i = base + threadIdx.x;
            const uint32_t c = i < nl ? ld_agent(&zt.cnt[i]) : 0u;
            uint32_t total = 0;
            const uint32_t ex = block_excl_scan<T>(c, total, red);
            if (i < nl) st_agent(&zt.off[i], run + ex);
            run += total;
        }
    }
    if (!csr_barrier(cc, ++b, nwg, timeout)) return false;
    // place each non-plain vertex in its level's group
    for (int64_t v = gtid; v < n; v += gsz) {
        if (!(ld_agent(&zt.flags[v]) & kNonPlain)) continue;
        const uint32_t L = ld_agent(&zt.lev[v]);
        const uint32_t pos = ld_agent(&zt.off[L]) +
                             __hip_atomic_fetch_add(&zt.fill[L], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        st_agent(&zt.seg[pos], (uint32_t)v);
    }
    if (!csr_barrier(cc, ++b, nwg, timeout)) return false;
    // the sequential pass of each level, a workgroup per level: settle the
    // lowest-index available vertex, make the heads of its tight zero-weight
    // edges available, repeat
    for (;;) {
        if (threadIdx.x == 0)
            claim = __hip_atomic_fetch_add(&cc->next_level, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __syncthreads();
        const uint32_t L = claim;
        __syncthreads();
        if (L >= nl) break;
        const uint32_t o = ld_agent(&zt.off[L]), cntL = ld_agent(&zt.cnt[L]);
        uint32_t pm = 0, step = 0;
        for (;;) {
            uint64_t best = kNoKey;
            for (uint32_t i = threadIdx.x; i < cntL; i += T) {
                const uint32_t v = ld_agent(&zt.seg[o + i]);
                const uint32_t f = ld_agent(&zt.flags[v]);
                if ((f & (kSeed | kAvail)) && !(f & kDone)) best = umin64(best, v);
            }
            uint32_t none = 0;
            block_min_or<T>(best, none, red);
            if (best == kNoKey) break;
            const uint32_t x = (uint32_t)best;
            pm = max(pm, x);
            ++step;
            if (threadIdx.x == 0) {
                set_flag(x, kDone);
                st_agent(&rk[x], ((uint64_t)pm << 32) | step);
            }
            const uint32_t dx = D(x);
            for (int64_t e = row_ptr[x] + threadIdx.x; e < row_ptr[x + 1]; e += T) {
                const int32_t y = col[e];
                if (w[e] == 0 && edge_ok((int32_t)x, y, 0, n) && D(y) == dx) set_flag(y, kAvail);
            }
            __builtin_amdgcn_s_waitcnt(0);
            __syncthreads();
        }
    }
    if (!csr_barrier(cc, ++b, nwg, timeout)) return false;
    // the smallest tail dist of a tight edge into each vertex ...
    for (int64_t u = gtid; u < n; u += gsz) {
        const uint32_t du = D(u);
        if (du >= kInf) continue;
        for_edges(row_ptr, col, w, n, (int32_t)u, [&](const int32_t* v, const int32_t* wt, const bool* eok) {
#pragma unroll
            for (int j = 0; j < kBatch; ++j)
                if (eok[j] && v[j] != src && tight(du, D(v[j]), wt[j]))
                    __hip_atomic_fetch_min(&zt.md[v[j]], du, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        });
    }
    if (!csr_barrier(cc, ++b, nwg, timeout)) return false;
    // ... the smallest settle key among those tails ...
    for (int64_t u = gtid; u < n; u += gsz) {
        const uint32_t du = D(u);
        if (du >= kInf) continue;
        const uint64_t ku = ld_agent(&rk[u]);
        for_edges(row_ptr, col, w, n, (int32_t)u, [&](const int32_t* v, const int32_t* wt, const bool* eok) {
#pragma unroll
            for (int j = 0; j < kBatch; ++j)
                if (eok[j] && v[j] != src && tight(du, D(v[j]), wt[j]) && ld_agent(&zt.md[v[j]]) == du)
                    __hip_atomic_fetch_min(&pk[v[j]], ku, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        });
    }
    if (!csr_barrier(cc, ++b, nwg, timeout)) return false;
    // ... and the tail whose key won is pred (one tail per vertex: keys differ within
    // a level); vertices without such a tail (the source, unreachable ones) get -1
    for (int64_t u = gtid; u < n; u += gsz) {
        const uint32_t du = D(u);
        if (du < kInf) {
            const uint64_t ku = ld_agent(&rk[u]);
            for_edges(row_ptr, col, w, n, (int32_t)u, [&](const int32_t* v, const int32_t* wt, const bool* eok) {
#pragma unroll
                for (int j = 0; j < kBatch; ++j)
                    if (eok[j] && v[j] != src && tight(du, D(v[j]), wt[j]) && ld_agent(&zt.md[v[j]]) == du &&
                        ld_agent(&pk[v[j]]) == ku)
                        pred[v[j]] = (int32_t)u;
            });
        }
        dist[u] = (int32_t)du;
        if (u == src || du >= kInf || ld_agent(&pk[u]) == kNoKey) pred[u] = -1;
    }
    return true;
}

template <int T>
__global__ __launch_bounds__(T) void k_csr_lc(const int64_t* __restrict__ row_ptr, const int32_t* __restrict__ col,
                                              const int32_t* __restrict__ w, int32_t n, int32_t src,
                                              int32_t* __restrict__ dist, int32_t* __restrict__ pred,
                                              uint64_t* __restrict__ lab, uint64_t* __restrict__ pkey,
                                              uint64_t* __restrict__ rk, uint32_t* __restrict__ lists,
                                              CsrCtl* __restrict__ cc, ZeroTie zt, long long team_limit,
                                              long long timeout, Ctl* __restrict__ ctl) {
    __shared__ Red<T> red;
    __shared__ SweepLds sl;
    const uint32_t rank = join_team(cc);
    if (rank & kTeamClosed) return;
    uint32_t b = 0, nwg = 0;
    unsigned long long sweeps = 0, rows = 0;
    uint32_t neg = 0;
    // distances: label-correcting sweeps from the source (the first frontier)
    bool ok = frontier_sweeps(
        rank, nwg, team_limit, cc->count, lists, lab, row_ptr, col, w, n, cc, b, timeout, 1u, sweeps, rows, sl,
        [&](int32_t u) { return label_value(ld_agent(&lab[u])); },
        [&](uint32_t du, int32_t u, int32_t v, int32_t wt, uint32_t& c) {
            if (!edge_ok(u, v, wt, n)) {
                neg |= wt < 0 ? 1u : 0u;
                return false;
            }
            c = du + (uint32_t)wt;  // both < 2^31: no wrap
            return c < kInf;        // longer than INT32_MAX - 1: not representable
        });
    const int64_t gtid = team_thread(rank, nwg);
    const int64_t gsz = (int64_t)nwg * T;
    uint32_t zero = 0;
    if (ok) {
        // pred pass: the tight edge of smallest (dist[u], u) into each vertex
        for (int64_t u = gtid; u < n; u += gsz) {
            const uint32_t du = label_value(ld_agent(&lab[u]));
            if (du >= kInf) continue;
            for_edges(row_ptr, col, w, n, (int32_t)u, [&](const int32_t* v, const int32_t* wt, const bool* eok) {
                uint32_t dv[kBatch];
#pragma unroll
                for (int j = 0; j < kBatch; ++j) dv[j] = eok[j] ? label_value(ld_agent(&lab[v[j]])) : kInf;
#pragma unroll
                for (int j = 0; j < kBatch; ++j) {
                    // unreachable heads have no pred
                    if (dv[j] >= kInf || du + (uint32_t)wt[j] != dv[j]) continue;
                    __hip_atomic_fetch_min(&pkey[v[j]], make_key(du, (uint32_t)u), __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_AGENT);
                    zero |= wt[j] == 0 ? 1u : 0u;
                }
            });
        }
        if (zero) __hip_atomic_fetch_or(&cc->zero, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (neg) __hip_atomic_fetch_or(&cc->neg, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        ok = csr_barrier(cc, ++b, nwg, timeout);
    }
    uint32_t status = ok ? 0u : kStatusTimeout;
    const uint32_t Z = ok ? ld_agent(&cc->zero) : 0u;
    if (ok && Z) {
        // tight zero-weight edges: the settle order of equal distances decides pred
        ok = zero_tie_pred<T>(rank, nwg, row_ptr, col, w, n, src, lab, rk, pkey, zt, cc, b, timeout, dist, pred, red);
        status |= ok ? kStatusZeroFallback : kStatusTimeout;
    } else if (ok) {
        for (int64_t v = gtid; v < n; v += gsz) {
            const uint32_t d = label_value(ld_agent(&lab[v]));
            const uint64_t kk = ld_agent(&pkey[v]);
            dist[v] = (int32_t)d;
            pred[v] = (v == src || d >= kInf || kk == kNoKey) ? -1 : (int32_t)(uint32_t)kk;
        }
    }
    if (rank == 0 && threadIdx.x == 0) {
        if (ok && ld_agent(&cc->neg)) status |= kStatusNegWeight;
        ctl->last[kStatRounds] = sweeps;
        ctl->last[kStatSettled] = rows;
        ctl->last[kStatFallbacks] = (status & kStatusZeroFallback) ? 1 : 0;
        ctl->last[kStatBarriers] = b + 1;
        ctl->status = status;
    }
}

}  // namespace

int csr_occupancy(int* per_cu) {
    return (int)hipOccupancyMaxActiveBlocksPerMultiprocessor(
        per_cu, reinterpret_cast<const void*>(&k_csr_lc<kCsrThreads>), kCsrThreads, 0);
}

}  // namespace sssp

using namespace sssp;

namespace {

// Workgroups of a CSR solve: about 256 vertices each, at most 1024 and at most the
// occupancy query times the compute units that no server's kernel holds (it can hold
// them for as long as queries come; close_team sees to what comes after this count).
// Beside a kernel on more than three quarters of them the hardware starts no workgroup
// until it leaves, and then they are all free.
// 1024 threads, one workgroup per CU: as many waves as 1024 workgroups of 256 threads
// with a quarter of the barrier's arrivals and of the appends' counter updates
// (n=10000: 174 us against 196 with 512 vertices each and 241 with 1024).
constexpr int kCsrMaxGrid = 1024;

int csr_grid(int32_t n, const sssp_tuning* tuning, int cus, int* nwg, int* per_cu_out) {
    int per_cu = 0;
    if (csr_occupancy(&per_cu) != 0 || per_cu < 1) return err(SSSP_EDEVICE, "CSR kernel does not fit a CU");
    int g = tuning && tuning->workgroups ? tuning->workgroups : (int)std::max<int64_t>(1, ((int64_t)n + 255) / 256);
    int dev = 0;
    (void)hipGetDevice(&dev);
    const int served = served_workgroups(dev);
    const int room = 4 * served <= 3 * cus ? cus - served : cus;
    *nwg = std::max(1, std::min({g, per_cu * room, kCsrMaxGrid}));
    if (per_cu_out) *per_cu_out = per_cu;
    return SSSP_OK;
}

}  // namespace

extern "C" {

int sssp_csr_grid(int32_t n, const sssp_tuning* tuning, void* stream, int32_t* workgroups, int32_t* per_cu,
                  int32_t* cus) {
    if (n < 1 || !workgroups) return err(SSSP_EINVAL, "bad arguments (n=%d)", n);
    Ctl* ctl = nullptr;
    int c = 0;
    long long khz = 0;
    int rc = stream_ctl((hipStream_t)stream, &ctl, &c, &khz);
    if (rc) return rc;
    int g = 0, pc = 0;
    if ((rc = csr_grid(n, tuning, c, &g, &pc))) return rc;
    *workgroups = g;
    if (per_cu) *per_cu = pc;
    if (cus) *cus = c;
    return SSSP_OK;
}

// Six launches and one copy back.  Against cursor atomics, a thread a row in the
// sort, seven launches and two copies: n=10000, m=3n, undirected 156 -> 85 us, 40000
// 165 -> 95 (sort 32 -> 9, fill 14 -> 8), 10^6 860 -> 660 (degrees 241 and fill 224,
// bound by scattered atomics and stores, sort 70); n=200000, m=16n 2660 -> 681.
int sssp_edges_to_csr(const int32_t* eu, const int32_t* ev, const int32_t* ew, int64_t m, int32_t n,
                      int32_t directed, int64_t* row_ptr, int32_t* col, int32_t* w, int64_t* m_out,
                      int64_t* bad_edges, void* stream) {
    if (!row_ptr || n < 1 || m < 0 || (m > 0 && (!eu || !ev || !ew || !col || !w)))
        return err(SSSP_EINVAL, "bad arguments (n=%d m=%lld)", n, (long long)m);
    hipStream_t s = (hipStream_t)stream;
    // scratch: the two counts and the degrees, which start at zero, the totals of the
    // scan's chunks, then each edge's places; where that is too much, cursors instead
    const int32_t chunks = (int32_t)(((int64_t)n + kScanChunk - 1) / kScanChunk);
    const size_t head = sizeof(unsigned long long) * (2 + (size_t)chunks), per_n = sizeof(uint32_t) * (size_t)n;
    const size_t ranks = sizeof(uint32_t) * (directed ? 1 : 2) * (size_t)m;
    char* buf = nullptr;
    bool ranked = true;
    hipError_t e = hipMallocAsync((void**)&buf, head + per_n + ranks, s);
    if (e != hipSuccess && ranks > per_n) {
        (void)hipGetLastError();
        ranked = false;
        e = hipMallocAsync((void**)&buf, head + 2 * per_n, s);
    }
    if (e != hipSuccess) return err(SSSP_ENOMEM, "hipMallocAsync: %s", hipGetErrorString(e));
    ConvertScratch cs{};
    cs.sums = reinterpret_cast<unsigned long long*>(buf);
    cs.out = cs.sums + chunks;
    cs.deg = reinterpret_cast<uint32_t*>(cs.out + 2);
    (ranked ? cs.rank : cs.cursor) = cs.deg + n;
    e = zero_fill(cs.out, 2 * sizeof(unsigned long long) + (ranked ? per_n : 2 * per_n), s);
    const unsigned eb = (unsigned)std::min<int64_t>(std::max<int64_t>(1, (m + 255) / 256), 8192);
    const unsigned nb = (unsigned)std::min<int64_t>(((int64_t)n + 31) / 32, 8192);
    if (e == hipSuccess && m > 0) {
        hipLaunchKernelGGL(k_csr_degree, dim3(eb), dim3(256), 0, s, eu, ev, ew, m, n, directed, cs);
        e = hipGetLastError();
    }
    if (e == hipSuccess) {
        const bool direct = chunks <= kScanDirect;
        hipLaunchKernelGGL(k_csr_chunk_sums, dim3(chunks), dim3(kScanChunk), 0, s, cs.deg, n, cs.sums);
        if (!direct) hipLaunchKernelGGL(k_csr_scan_sums, dim3(1), dim3(kScanChunk), 0, s, cs.sums, chunks);
        hipLaunchKernelGGL(k_csr_scan_chunks, dim3(chunks), dim3(kScanChunk), 0, s, cs.deg, n, cs.sums, direct, row_ptr,
                           cs.out + 1);
        e = hipGetLastError();
    }
    if (e == hipSuccess && m > 0) {
        hipLaunchKernelGGL(k_csr_fill, dim3(eb), dim3(256), 0, s, eu, ev, ew, m, n, directed, row_ptr, cs, col, w);
        e = hipGetLastError();
    }
    if (e == hipSuccess && m > 0) {
        hipLaunchKernelGGL(k_csr_sort_rows, dim3(nb), dim3(256), 0, s, row_ptr, n, col, w);
        e = hipGetLastError();
    }
    unsigned long long out[2] = {0, 0};
    if (e == hipSuccess) e = hipMemcpyAsync(out, cs.out, sizeof out, hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    (void)hipFreeAsync(buf, s);
    if (e != hipSuccess) return err(SSSP_EDEVICE, "edge list conversion: %s", hipGetErrorString(e));
    if (m_out) *m_out = (int64_t)out[1];
    if (bad_edges) *bad_edges = (int64_t)out[0];
    return SSSP_OK;
}

int sssp_csr_solve(const int64_t* row_ptr, const int32_t* col, const int32_t* w, int32_t n, int32_t src,
                   int32_t* dist, int32_t* pred, const sssp_tuning* tuning, void* stream) {
    if (!row_ptr || !dist || !pred || n < 1) return err(SSSP_EINVAL, "bad arguments (n=%d)", n);
    if (src < 0 || src >= n) return err(SSSP_EINVAL, "src %d outside [0, %d)", src, n);
    hipStream_t s = (hipStream_t)stream;
    Ctl* ctl = nullptr;
    int cus = 0;
    long long khz = 100000;
    int rc = stream_ctl(s, &ctl, &cus, &khz);
    if (rc) return rc;
    int nwg = 0;
    if ((rc = csr_grid(n, tuning, cus, &nwg, nullptr))) return rc;
    // scratch: dist labels, pred keys, settle keys (n x 8 B each), 3 frontier lists
    // (3n words), control, and the tables of the zero-weight tie pass (7n words,
    // 12 B per entry of a table of the smallest power of two >= 2n entries)
    const size_t words = (size_t)n;
    uint32_t hbits = 1;
    while ((1ull << hbits) < 2ull * words) ++hbits;
    const size_t H = (size_t)1 << hbits;
    const size_t bytes = 3 * words * 8 + 3 * words * 4 + sizeof(CsrCtl) + 256 + H * 8 + 7 * words * 4 + H * 4 + 256;
    char* buf = nullptr;
    hipError_t e = hipMallocAsync((void**)&buf, bytes, s);
    if (e != hipSuccess) return err(SSSP_ENOMEM, "hipMallocAsync(%zu bytes): %s", bytes, hipGetErrorString(e));
    uint64_t* lab = reinterpret_cast<uint64_t*>(buf);
    uint64_t* pkey = lab + words;
    uint64_t* rk = pkey + words;
    uint32_t* lists = reinterpret_cast<uint32_t*>(rk + words);
    CsrCtl* cc = reinterpret_cast<CsrCtl*>(((uintptr_t)(lists + 3 * words) + 255) & ~(uintptr_t)255);
    ZeroTie zt;
    zt.ht_key = reinterpret_cast<uint64_t*>(((uintptr_t)(cc + 1) + 255) & ~(uintptr_t)255);
    zt.ht_lvl = reinterpret_cast<uint32_t*>(zt.ht_key + H);
    zt.flags = zt.ht_lvl + H;
    zt.lev = zt.flags + words;
    zt.seg = zt.lev + words;
    zt.cnt = zt.seg + words;
    zt.off = zt.cnt + words;
    zt.fill = zt.off + words;
    zt.md = zt.fill + words;
    zt.hbits = hbits;
    const unsigned ib = (unsigned)std::min<int64_t>((n + 255) / 256, 4096);
    hipLaunchKernelGGL(k_csr_init, dim3(ib), dim3(256), 0, s, n, src, row_ptr, w, lab, pkey, lists, cc);
    e = hipGetLastError();
    if (e == hipSuccess) {
        long long timeout = grid_barrier_ticks(khz);
        long long limit = std::min(timeout, khz * kTeamWaitUs / 1000);
#ifdef SSSP_STRESS_DELAYS
        limit /= 40;  // some arrive too late
#endif
        if (grid_launch_is_plain()) {
            // ordinary launch of the same grid (co-resident by its size), for profilers
            hipLaunchKernelGGL(k_csr_lc<kCsrThreads>, dim3(nwg), dim3(kCsrThreads), 0, s, row_ptr, col, w, n, src,
                               dist, pred, lab, pkey, rk, lists, cc, zt, limit, timeout, ctl);
            e = hipGetLastError();
        } else {
            void* args[] = {(void*)&row_ptr, (void*)&col, (void*)&w, &n, &src, &dist, &pred, &lab, &pkey,
                            &rk, &lists, &cc, &zt, &limit, &timeout, &ctl};
            e = hipLaunchCooperativeKernel(reinterpret_cast<const void*>(&k_csr_lc<kCsrThreads>), dim3(nwg),
                                           dim3(kCsrThreads), args, 0, s);
        }
    }
    (void)hipFreeAsync(buf, s);
    if (e != hipSuccess) return err(SSSP_EDEVICE, "CSR solve launch: %s", hipGetErrorString(e));
    return SSSP_OK;
}

}  // extern "C"
