// Label-correcting solve: the paper's CUDA design (Section III-C, Algorithms 3
// and 4) made deterministic and coalesced.  The single-solve call offers it as
// an alternative to the Dijkstra rounds; batched plans and servers use it for
// graphs whose solves need many rounds (sparse graphs with many distinct
// distances), where it replaces hundreds of exchanges by a few sweeps.
//
// Algorithm 4 lets every vertex relax its whole row in each sweep, with an
// atomicMin on dist and a separate, racy store of pred, and Algorithm 3 repeats
// sweeps until no dist changes.  Here:
//   * a sweep relaxes only the rows of the vertices whose dist changed in the
//     previous sweep (the frontier; the first frontier is the source), each row
//     with the dist its vertex had when the sweep started;
//   * every workgroup owns a column slice, as in the whole-GPU Dijkstra solve,
//     so the per-column minimum needs no atomics and the rows are read by
//     consecutive lanes (coalesced) rather than one row per thread;
//   * the convergence test is on the device: a sweep whose frontier is empty
//     ends the loop, with no host round trip;
//   * pred is not written during the sweeps, but the rows are read only in them:
//     beside the smallest dist(u) + W[u][v] offered to column v, each thread keeps
//     the lexicographically smallest (dist(u), u) that offered it, u != v.  Every
//     reachable u is relaxed with its final dist in the sweep after that dist was
//     found, and an offer made with a larger one is larger than v's final dist, so
//     once dist is final the kept u is the smallest with dist(u) + W[u][v] ==
//     dist[v].  When no such tight edge has weight 0, Algorithm 1 settles vertices
//     in (dist, index) order, and that u is the first settled vertex to offer
//     dist[v] — exactly the pred its strict '<' keeps.  If a tight zero-weight edge
//     (u != v) was offered, the order of Algorithm 1 is no longer (dist, index), so
//     the launch re-solves with the Dijkstra rounds instead (status bit
//     ZERO_FALLBACK).  (A last pass over all rows for pred took 84 of 441 us at
//     n=8192, p=0.001.)
// dist is exact in every case: it is the unique shortest-path distance, which
// any label-correcting order reaches.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "engine.h"
#include "solve.h"

namespace sssp {

// LDS beyond SharedSolve: dist of the staged frontier rows, and the columns'
// dist, to which the row partitions merge what they found in a sweep.
template <int T>
struct SharedLC {
    uint32_t dl[kCap];
    uint32_t dcol[4 * T];
};
template <int T>
__shared__ SharedLC<T> g_lc;

// A frontier entry is one word: the vertex's dist (31 bits), its column in the
// member's slice (14 bits: a slice has at most 16384) and the low bits of the tag
// of its exchange (see tag_word); bit 63 stays clear (see exchange_stamp).
constexpr int kLcColShift = 31, kLcTagShift = 45;
constexpr int kLcTagBits = 18;
constexpr uint32_t kLcTagMask = (1u << kLcTagBits) - 1u;
__host__ __device__ constexpr uint64_t lc_word(uint32_t tag, uint32_t col, uint32_t d) {
    return ((uint64_t)(tag & kLcTagMask) << kLcTagShift) | ((uint64_t)col << kLcColShift) | d;
}
__host__ __device__ constexpr uint32_t lc_word_tag(uint64_t w) { return (uint32_t)(w >> kLcTagShift); }
__host__ __device__ constexpr uint32_t lc_word_col(uint64_t w) { return (uint32_t)(w >> kLcColShift) & 0x3fffu; }
__host__ __device__ constexpr uint32_t lc_word_dist(uint64_t w) { return (uint32_t)w & 0x7fffffffu; }

// A member's record of a sweep is two words of its rec_word line: the number of
// its entries (kLcCount, full tag) and the first of them (kLcFirst); the others
// are in its list from index 1 on.
enum { kLcCount = 0, kLcFirst = 1 };

// Loads of U rows (list[i], list[i + step], ...) of one column group, widened;
// past the end of the list the last row repeats (harmless for a minimum).
template <int U, typename E, bool NT>
__device__ __forceinline__ void lc_load(uint32_t (&w)[U][4], uint32_t (&uu)[U], uint32_t (&du)[U],
                                        const E* __restrict__ p0, int64_t ld, const int32_t* list,
                                        const uint32_t* dl, int m, int i, int step) {
#pragma unroll
    for (int q = 0; q < U; ++q) {
        const int idx = i + q * step;
        const int ii = idx < m ? idx : m - 1;
        uu[q] = (uint32_t)list[ii];
        du[q] = dl[ii];
    }
    typename Raw<E>::type raw[U];
#pragma unroll
    for (int q = 0; q < U; ++q) {
        const global_ptr<typename Raw<E>::type> a =
            reinterpret_cast<global_ptr<typename Raw<E>::type>>((global_ptr<E>)p0 + (int64_t)uu[q] * ld);
        raw[q] = NT ? __builtin_nontemporal_load(a) : *a;
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int q = 0; q < U; ++q) {
        unpack<E>(raw[q], w[q]);
#pragma unroll
        for (int j = 0; j < 4; ++j) w[q][j] = widen<E>(w[q][j]);  // compact codes -> weights
    }
}

// What a column keeps of a tail u of dist du: compares as (du, u), above kZeroTight.
constexpr uint64_t kZeroTight = 0;  // a tight edge of weight 0 (from u != v) was among the offers
__host__ __device__ constexpr uint64_t lc_entry(uint32_t d, uint32_t v) { return ((uint64_t)d << 32) | v; }
__device__ __forceinline__ uint64_t lc_key(uint32_t du, uint32_t u) { return lc_entry(du, u) + 1; }

// c = du + w, clamped, offered by row u to column v: best and the key of who
// offered it.
__device__ __forceinline__ void lc_offer(uint32_t& best, uint64_t& key, uint32_t c, uint32_t du, uint32_t u,
                                         uint32_t w, uint32_t v) {
    if (c > best || c >= kInf) return;
    const uint64_t k = w == 0u && u != v ? kZeroTight : lc_key(du, u);
    key = c < best ? k : umin64(key, k);
    best = c;
}

// U staged rows of one column group.  No edge (INT32_MAX) and negative weights (>
// INT32_MAX as uint32) offer nothing: their clamped sums are at least INT32_MAX,
// which no best exceeds.  neg collects the weights' sign bits.  Few rows of a sparse
// graph offer a thread's columns anything, so a row's four offers share one branch
// (three operations an entry beside the loads; with the tests for no edge and for a
// sign on each entry seven).
template <int U, typename E, bool NT>
__device__ __forceinline__ void lc_batch(uint32_t (&best)[4], uint64_t (&key)[4], uint32_t v0,
                                         const E* __restrict__ p0, int64_t ld, const int32_t* list,
                                         const uint32_t* dl, int m, int i, int step, uint32_t& neg) {
    uint32_t w[U][4], uu[U], du[U];
    lc_load<U, E, NT>(w, uu, du, p0, ld, list, dl, m, i, step);
#pragma unroll
    for (int q = 0; q < U; ++q) {
        uint32_t c[4];
        bool any = false;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            c[j] = __builtin_elementwise_add_sat(du[q], w[q][j]);
            any |= c[j] <= best[j];
        }
        if (sizeof(E) == 4) neg |= w[q][0] | w[q][1] | w[q][2] | w[q][3];
        if (any)
#pragma unroll
            for (int j = 0; j < 4; ++j) lc_offer(best[j], key[j], c[j], du[q], uu[q], w[q][j], v0 + (uint32_t)j);
    }
}

// The staged rows first, first + step, ...: few in a batch of their size, as in
// stream_group.
template <int U, typename E, bool NT>
__device__ __forceinline__ void lc_sweep_group(uint32_t (&best)[4], uint64_t (&key)[4], uint32_t v0,
                                               const E* __restrict__ p0, int64_t ld, const int32_t* list,
                                               const uint32_t* dl, int m, int first, int step, uint32_t& neg) {
    if (m <= 2 * step) {
        if (first >= m) return;
        if (m <= step) lc_batch<1, E, NT>(best, key, v0, p0, ld, list, dl, m, first, step, neg);
        else lc_batch<2, E, NT>(best, key, v0, p0, ld, list, dl, m, first, step, neg);
        return;
    }
    for (int i = first; i < m; i += step * U) lc_batch<U, E, NT>(best, key, v0, p0, ld, list, dl, m, i, step, neg);
}

// One pass of the staged rows over this thread's column groups (partial last
// groups as in stream_rows).
template <int G, int U, typename E, bool NT>
__device__ __forceinline__ void lc_sweep_rows(uint32_t (&best)[G][4], uint64_t (&key)[G][4], const Layout& lo,
                                              const E* __restrict__ W, int64_t ld, int64_t col0, int width,
                                              const int32_t* list, const uint32_t* dl, int m, uint32_t& neg) {
#pragma unroll
    for (int k = 0; k < G; ++k) {
        const int v0 = 4 * (lo.c + k * lo.L);
        if (v0 >= width) continue;
        const int s = group_shift<E>(v0, width);
        if (col0 + v0 < s) {  // a matrix of fewer than 4 columns
            for (int i = lo.r; i < m; i += lo.P)
                for (int j = 0; j < 3; ++j) {
                    const uint32_t w = j < width ? widen<E>((uint32_t)W[(int64_t)list[i] * ld + j]) : kInf;
                    neg |= w;
                    lc_offer(best[k][j], key[k][j], __builtin_elementwise_add_sat(dl[i], w), dl[i],
                             (uint32_t)list[i], w, (uint32_t)j);
                }
            continue;
        }
        if (s) {  // a neighbour's column, dropped afterwards, takes no offers
            shift_up(best[k], s, 0u);
            shift_up(key[k], s, kNoKey);
        }
        lc_sweep_group<U, E, NT>(best[k], key[k], (uint32_t)(col0 + v0 - s), W + (col0 + v0 - s), ld, list, dl, m,
                                 lo.r, lo.P, neg);
        if (s) {
            shift_down(best[k], s, 0u);
            shift_down(key[k], s, kNoKey);
        }
    }
}

// Merge what the P row partitions found in a sweep (P > 1 implies G == 1): those
// that lowered a column tell dcol, the columns' dist, and all go on from it, a
// partition's key being of use only while its best is the column's.
template <int T, int G>
__device__ __forceinline__ void lc_merge(uint32_t (&best)[G][4], uint64_t (&key)[G][4], const uint32_t (&old)[G][4],
                                         const Layout& lo, uint32_t* dcol) {
    if (lo.P == 1) return;
#pragma unroll
    for (int j = 0; j < 4; ++j)
        if (best[0][j] < old[0][j])
            __hip_atomic_fetch_min(&dcol[j * lo.L + lo.c], best[0][j], __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_WORKGROUP);
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const uint32_t d = dcol[j * lo.L + lo.c];
        if (d < best[0][j]) {
            best[0][j] = d;
            key[0][j] = kNoKey;
        }
    }
}

// Merge the row partitions' keys into the owners (partition 0) with LDS atomic
// minima, as merge_partitions does (the merge area is all ones between merges).
template <int T, int G>
__device__ __forceinline__ void lc_merge_keys(uint64_t (&key)[G][4], const Layout& lo, uint64_t* mrg) {
    if (lo.P == 1) return;
#pragma unroll
    for (int j = 0; j < 4; ++j)
        if (key[0][j] != kNoKey)
            __hip_atomic_fetch_min(&mrg[j * lo.L + lo.c], key[0][j], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    __syncthreads();
    if (lo.r == 0) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            key[0][j] = mrg[j * lo.L + lo.c];
            mrg[j * lo.L + lo.c] = kNoKey;
        }
    }
}

// Publish the owned columns selected by `mask` as entries of exchange `tag`, with
// their count.  Nothing waits for the stores: readers check each word's tag.  An
// entry's tag has fewer bits than the exchange number, and a slot of a list can
// hold an entry from long ago: every half period the member first gives its words of
// the slot the tag of exchange tag - 2, the last one in it, which all have read.
template <int T, int G>
__device__ __forceinline__ void lc_publish(uint32_t mask, const uint32_t (&dv)[G][4], const Layout& lo, uint32_t tag,
                                           uint64_t* __restrict__ recs, int nwg, int g, uint64_t* __restrict__ list,
                                           int S, SharedSolve<T>& sh) {
    uint64_t* rec = rec_word(recs, nwg, (tag - 1) & 1, 0, g);
    if ((tag & (kLcTagMask >> 1) & ~1u) == 0 && tag > 1) {
        for (int i = threadIdx.x; i < S; i += T) st_agent(&list[i], lc_word(tag - 2, 0, 0));
        if (threadIdx.x == 0) st_agent(&rec[kLcFirst], lc_word(tag - 2, 0, 0));
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
    }
    uint32_t total = 0;
    uint32_t rank = owner_excl_scan<T>(__popc(mask), total, lo.L, sh.red);
    if (mask) stress_delay(2u * tag + 1u);
#pragma unroll
    for (int k = 0; k < G; ++k)
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (mask >> (4 * k + j) & 1u) {
                st_agent(rank ? &list[rank] : &rec[kLcFirst], lc_word(tag, (uint32_t)local_col(lo, k, j), dv[k][j]));
                ++rank;
            }
    if (threadIdx.x == 0) {
        stress_delay(2u * tag);
        st_agent(&rec[kLcCount], tag_word(tag, total));
    }
}

// Position p of an exchange's concatenated entries belongs to this member: wave 0
// reads gangs of up to 256 members, lane l taking l, l + 64, l + 128 and l + 192.
__device__ __forceinline__ int lc_member(int p, int nwg) { return nwg <= 4 * kWave ? (p >> 2) + kWave * (p & 3) : p; }

// Exchange `tag` from the reader's side: waits for the members' counts and first
// entries, leaves the counts' offsets in sh.pre (by position) and returns their sum.
// When no member has a second entry the frontier is staged in sh.list / lc.dl here,
// and *staged tells (as in read_records).  *late: a word did not arrive in time.
template <int T, int KM>
__device__ __forceinline__ void lc_read_wave(uint64_t* recs, int S, int nwg, uint32_t tag, long long timeout,
                                             SharedSolve<T>& sh, SharedLC<T>& lc) {
    const int l = wave_lane();
    uint32_t late = sh.stage_late;
    uint64_t a[KM], e[KM];
    long long t0 = 0;
    unsigned naps = 0;
    for (;;) {
        // all loads issued before any is used (member indexes clamped)
#pragma unroll
        for (int k = 0; k < KM; ++k) {
            const uint64_t* w = rec_word(recs, nwg, (tag - 1) & 1, 0, min(l + kWave * k, nwg - 1));
            a[k] = ld_agent(&w[kLcCount]);
            e[k] = ld_agent(&w[kLcFirst]);
        }
        bool there = true;
#pragma unroll
        for (int k = 0; k < KM; ++k)
            there = there && word_tag(a[k]) == tag &&
                    ((uint32_t)a[k] == 0u || lc_word_tag(e[k]) == (tag & kLcTagMask));
        if (!wave_mask(!there) || late) break;
        const long long now = wall_clock64();
        if (t0 == 0) t0 = now;
        if (now - t0 >= timeout) {
            late = 1;
            break;
        }
        for (unsigned i = 0; i < naps; ++i) __builtin_amdgcn_s_sleep(1);
        naps = naps ? (naps < 4 ? naps << 1 : naps) : 1;
    }
    late = wave_mask(late != 0) ? 1u : 0u;
    uint32_t c[KM], local = 0, most = 0;
#pragma unroll
    for (int k = 0; k < KM; ++k) {
        c[k] = l + kWave * k < nwg && !late ? (uint32_t)a[k] : 0u;
        local += c[k];
        most = max(most, c[k]);
    }
    const uint32_t inc = wave_prefix32(local);
    uint32_t run = inc - local;
    const bool small = wave_mask(most > 1u) == 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const uint32_t ck = k < KM ? c[k < KM ? k : 0] : 0u;
        const uint64_t ek = e[k < KM ? k : 0];
        sh.pre[4 * l + k] = run;
        if (small && ck) {
            sh.list[run] = (l + kWave * k) * S + (int)lc_word_col(ek);
            lc.dl[run] = lc_word_dist(ek);
        }
        run += ck;
    }
    if (l == kWave - 1) {
        sh.res[tag & 1u].rows = inc;
        sh.res[tag & 1u].flags = (small ? 2u : 0u) | (late << 2);
    }
}

template <int T>
__device__ __forceinline__ uint32_t lc_records(uint64_t* recs, int S, int nwg, uint32_t tag, long long timeout,
                                               SharedSolve<T>& sh, SharedLC<T>& lc, bool& staged, bool& ok) {
    if (nwg <= 4 * kWave) {
        if (threadIdx.x < kWave) {
            if (nwg <= kWave) lc_read_wave<T, 1>(recs, S, nwg, tag, timeout, sh, lc);
            else lc_read_wave<T, 4>(recs, S, nwg, tag, timeout, sh, lc);
        }
        __syncthreads();
        const uint32_t z = scalar(sh.res[tag & 1u].flags);
        staged = (z & 2u) != 0;
        ok = (z & 4u) == 0;
        return scalar(sh.res[tag & 1u].rows);
    }
    uint32_t c = 0, late = sh.stage_late;
    if ((int)threadIdx.x < nwg) {
        const uint64_t* w = rec_word(recs, nwg, (tag - 1) & 1, 0, (int)threadIdx.x);
        c = (uint32_t)wait_tag(&w[kLcCount], ld_agent(&w[kLcCount]), tag, timeout, late);
    }
    uint64_t dummy = kNoKey;
    block_min_or<T>(dummy, late, sh.red);
    ok = late == 0;
    staged = false;
    uint32_t M;
    const uint32_t pre = block_excl_scan<T>(ok ? c : 0u, M, sh.red);
    if ((int)threadIdx.x < nwg) sh.pre[threadIdx.x] = pre;
    __syncthreads();
    return M;
}

// Entry e0 + threadIdx.x of the concatenated lists: its vertex and dist.
template <int T>
__device__ __forceinline__ void lc_gather(SharedSolve<T>& sh, uint64_t* recs, const uint64_t* __restrict__ rl,
                                          int nwg, int S, uint32_t tag, long long timeout, uint32_t e0, uint32_t M,
                                          int32_t& v, uint32_t& d) {
    v = 0;
    d = 0;
    const uint32_t e = e0 + threadIdx.x;
    if (e >= M) return;
    int lo_i = 0, hi_i = nwg <= 4 * kWave ? 4 * kWave - 1 : nwg - 1;
    while (lo_i < hi_i) {
        const int mid = (lo_i + hi_i + 1) >> 1;
        if (sh.pre[mid] <= e) lo_i = mid;
        else hi_i = mid - 1;
    }
    const int m = lc_member(lo_i, nwg);
    const uint32_t at = e - sh.pre[lo_i];
    const uint64_t* p = at ? &rl[(size_t)m * S + at] : rec_word(recs, nwg, (tag - 1) & 1, kLcFirst, m);
    uint64_t w = ld_agent(p);
    if (lc_word_tag(w) != (tag & kLcTagMask)) {
        const long long t0 = wall_clock64();
        do {
            __builtin_amdgcn_s_sleep(1);
            w = ld_agent(p);
            if (wall_clock64() - t0 > timeout) {  // a valid row; the solve then ends with the time-out status
                sh.stage_late = 1;
                v = m * S;
                return;
            }
        } while (lc_word_tag(w) != (tag & kLcTagMask));
    }
    v = m * S + (int)lc_word_col(w);
    d = lc_word_dist(w);
}

// Stage the M listed rows chunk by chunk into LDS (unless lc_records has) and run
// `pass` over each chunk; the next chunk's entries load while the current one streams.
template <int T, class Pass>
__device__ __forceinline__ void lc_stream(uint64_t* recs, const uint64_t* rl, int nwg, int S, uint32_t tag,
                                          long long timeout, uint32_t M, bool staged, SharedSolve<T>& sh,
                                          SharedLC<T>& lc, Pass pass) {
    if (staged) {
        pass((int)M);
        __syncthreads();
        return;
    }
    int32_t v;
    uint32_t d;
    lc_gather<T>(sh, recs, rl, nwg, S, tag, timeout, 0, M, v, d);
    for (uint32_t e0 = 0; e0 < M; e0 += kCap) {
        sh.list[threadIdx.x] = v;
        lc.dl[threadIdx.x] = d;
        __syncthreads();
        if (e0 + kCap < M) lc_gather<T>(sh, recs, rl, nwg, S, tag, timeout, e0 + kCap, M, v, d);
        pass((int)min((uint32_t)kCap, M - e0));
        __syncthreads();
    }
}

enum LcResult { kLcDone = 0, kLcTimeout = 1, kLcFallback = 2 };

// Rank g of a gang of nwg workgroups (the whole grid), with the exchange memory gw
// of the Dijkstra rounds: stamped records for the first exchange, which tells that
// every member has cleared its tagged words, and for the last, after which nobody
// reads them; tagged records and lists, double-buffered by exchange parity, for the
// sweeps.  b counts the exchanges passed (a fallback solve continues the numbering);
// epoch stamps this launch's records (see gang_exchange).  Small sweeps are bound by
// the exchange: with stamped records (store, wait, stamp, poll, read the records, read
// the entries) and eight loads of a single row one of a few rows took 4.9 us on 256
// workgroups, with tagged words and loads as needed 3.3.  (Whole solves, n=8192,
// p=0.001: 405 us with a pass for pred, 352 without it, 289 with the rest.)
template <int T, int G, int U, typename E, bool NT>
__device__ __forceinline__ int solve_lc(const E* __restrict__ W, int64_t ld, int32_t n, int32_t src,
                                        int32_t* __restrict__ dist, int32_t* __restrict__ pred, int S,
                                        int g, int nwg, long long timeout, const GangWords& gw,
                                        SharedSolve<T>& sh, SharedLC<T>& lc, SolveStats& st, uint32_t& b,
                                        uint32_t epoch, Ctl* trace) {
    static_assert(T == kCap, "one staged entry per thread");
    const int64_t col0 = (int64_t)g * S;
    const int width = (int)max((int64_t)0, min((int64_t)S, (int64_t)n - col0));
    const Layout lo = make_layout<T>(S);
    uint32_t dv[G][4];   // dist of the thread's columns: the owners' as the members know it
    uint64_t key[G][4];  // who offered it to this partition (kNoKey: nobody)
    uint32_t own = 0;
#pragma unroll
    for (int k = 0; k < G; ++k)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int v = local_col(lo, k, j);
            const bool is_src = k * lo.L + lo.c < lo.NG && v < width && col0 + v == src;
            const bool mine = lo.r == 0 && k * lo.L + lo.c < lo.NG && v < width;
            dv[k][j] = is_src ? 0u : kInf;
            key[k][j] = kNoKey;
            own |= mine ? 1u << (4 * k + j) : 0u;
            if (lo.P > 1 && lo.r == 0) lc.dcol[j * lo.L + lo.c] = dv[k][j];
        }
    clear_merge<T>(sh.mrg, 4 * T);
    if (threadIdx.x == 0) sh.stage_late = 0;
    clear_tagged<T>(gw.recs, gw.lists, gw.ctr, gw.done, g, nwg, S);
    // the stamped exchanges: members' records of slot (b & 1) carry stamp b + 1
    auto slot_pub = [&](uint32_t s) { return gw.pubs + (size_t)s * nwg; };
    auto exchange = [&]() {
        ++b;
        return gang_exchange<T>(slot_pub((b - 1) & 1), g, exchange_stamp(epoch, b), (uint32_t)nwg, timeout, sh.red);
    };
    if (!exchange()) return kLcTimeout;

    // sweep 1 relaxes the source's row
    uint32_t M = 1;
    bool staged = true, ok = true;
    if (threadIdx.x == 0) {
        sh.list[0] = src;
        lc.dl[0] = 0;
    }
    __syncthreads();
    uint32_t neg = 0;
    while (M) {
        uint64_t* rl = gw.lists + (size_t)((b - 1) & 1) * nwg * S;
        ++st.rounds;
        st.settled += M;
        const long long t_round = wall_clock64();
        uint32_t old[G][4];
#pragma unroll
        for (int k = 0; k < G; ++k)
#pragma unroll
            for (int j = 0; j < 4; ++j) old[k][j] = dv[k][j];
        lc_stream<T>(gw.recs, rl, nwg, S, b, timeout, M, staged, sh, lc, [&](int m) {
            lc_sweep_rows<G, U, E, NT>(dv, key, lo, W, ld, col0, width, sh.list, lc.dl, m, neg);
        });
        lc_merge<T, G>(dv, key, old, lo, lc.dcol);
        if (trace && g == 0 && threadIdx.x == 0 && st.rounds <= (unsigned long long)kTraceCap) {
            trace->trace_t[st.rounds - 1] = t_round;
            trace->trace_m[st.rounds - 1] = M;
        }
        uint32_t chg = 0;
#pragma unroll
        for (int k = 0; k < G; ++k)
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if ((own >> (4 * k + j) & 1u) && dv[k][j] < old[k][j]) chg |= 1u << (4 * k + j);
        ++b;
        lc_publish<T, G>(chg, dv, lo, b, gw.recs, nwg, g, gw.lists + ((size_t)((b - 1) & 1) * nwg + g) * S, S, sh);
        M = lc_records<T>(gw.recs, S, nwg, b, timeout, sh, lc, staged, ok);
        if (!ok) break;
    }
    st.status |= neg >> 31 ? kStatusNegWeight : 0u;
    if (!ok) return kLcTimeout;

    lc_merge_keys<T, G>(key, lo, sh.mrg);
    uint32_t reach = 0, zero = 0;
#pragma unroll
    for (int k = 0; k < G; ++k)
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if ((own >> (4 * k + j) & 1u) && dv[k][j] < kInf) {
                ++reach;
                zero |= key[k][j] == kZeroTight ? 1u : 0u;
            }
    uint32_t reached = 0;
    (void)owner_excl_scan<T>(reach, reached, lo.L, sh.red);
    // agree on the tight-zero-edge verdict before writing anything
    uint64_t dummy = kNoKey;
    block_min_or<T>(dummy, zero, sh.red);
    if (threadIdx.x == 0) {
        Pub* p = &slot_pub(b & 1)[g];
        st_agent(&p->key, (uint64_t)0);
        st_agent(&p->count, reached);
        st_agent(&p->flags, zero);
    }
    if (!exchange()) return kLcTimeout;
    // the reachable vertices count a second time, as the rows a pass for pred would read
    uint32_t count = 0, Z = 0, all = 0;
    if ((int)threadIdx.x < nwg) {
        const Pub* p = &slot_pub((b - 1) & 1)[threadIdx.x];
        count = ld_agent(&p->count);
        Z = ld_agent(&p->flags);
    }
    (void)block_excl_scan<T>(count, all, sh.red);
    st.settled += all;
    block_min_or<T>(dummy, Z, sh.red);
    if (Z) return kLcFallback;
    if (lo.r == 0) {
#pragma unroll
        for (int k = 0; k < G; ++k)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if (!(own >> (4 * k + j) & 1u)) continue;
                const int64_t v = col0 + local_col(lo, k, j);
                dist[v] = (int32_t)dv[k][j];
                pred[v] = (v == src || dv[k][j] >= kInf || key[k][j] == kNoKey) ? -1 : (int32_t)(uint32_t)(key[k][j] - 1);
            }
    }
    return kLcDone;
}

}  // namespace sssp
