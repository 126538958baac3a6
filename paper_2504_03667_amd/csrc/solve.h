// Round engines shared by the kernels: one workgroup solving a whole instance
// (solve_single) and a gang of workgroups that each own a column slice and
// meet at one barrier per round (solve_gang), with the barrier, the per-round
// records and the bucket gather they use.  See kernels.hip for the method.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "engine.h"
#include "sssp_internal.h"

namespace sssp {

constexpr int kCap = 1024;  // bucket rows staged in LDS per chunk
constexpr int kSingleMax = 16384;  // vertices of the largest one-workgroup solve (4 groups of 4 x 1024 threads)
constexpr uint32_t kPairChunks = 8;  // chunks from which a round is balanced within pairs (solve_gang)
constexpr uint32_t kPairUnit = 256;  // rows per claim unit of a balanced round

template <int T>
struct SharedSolve {
    Red<T> red;
    union {
        int32_t list[kCap];
        uint16_t list16[kSingleMax];  // solve_single: the whole bucket
    };
    uint64_t mrg[4 * T];
    uint32_t pre[T];
    uint32_t cnt[T];
    // read_records results for the whole workgroup, by exchange parity.  A round in
    // which the slice reads no row has no barrier between the reads of one exchange's
    // result and wave 0's stores of the next: those go to the other slot, and wave 0
    // comes back to this one only after the next exchange's barrier, which every
    // wave passes after its reads.
    struct alignas(16) {
        uint32_t d, vert, rows, flags;
    } res[2];
    uint64_t res_need[2];  // ... and, for narrow slices, the lanes whose group the next round reads
    uint32_t claim[2];    // chunk claims of a balanced round, broadcast by thread 0
    uint32_t stage_late;  // a bucket entry did not arrive in time (set once; the solve then ends)
    int32_t item;
    uint32_t flag;
    uint64_t min3[3];    // solve_single: lowest key of a round, by round number mod 3; [0]: publish, wide slices
    uint32_t count3[3];  // ... and its bucket's size
    uint32_t open3[3];   // groups a round can lower, by round number mod 3 (also solve_gang)
    uint32_t listed;     // ... of a sparse round, how many are in group
    uint16_t group[kSparseGroups];  // ... and which (local column / 4)
    uint64_t sparse[4 * kSparseGroups];  // their keys in a sparse round, all ones between rounds
};

// The owners (the threads below L: whole waves, or lanes of wave 0) count the
// groups that a round at d can lower in open3[slot]; ordered before its readers by
// a workgroup barrier.
template <int T, int G>
__device__ __forceinline__ void count_groups(const uint32_t (&x)[G][4], uint32_t d, uint32_t wmin, uint32_t slot,
                                             SharedSolve<T>& sh) {
    uint32_t count = 0;
#pragma unroll
    for (int k = 0; k < G; ++k) count += (uint32_t)__popcll(wave_mask(group_open(x[k], d, wmin)));
    if (count && (threadIdx.x & (kWave - 1)) == 0)
        __hip_atomic_fetch_add(&sh.open3[slot], count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// ... and list a sparse round's in sh.group, in any order (sh.listed: zero before,
// and again afterwards by the caller).
template <int T, int G>
__device__ __forceinline__ void list_groups(const uint32_t (&x)[G][4], uint32_t d, uint32_t wmin, const Layout& lo,
                                            SharedSolve<T>& sh) {
    if (lo.r == 0)
#pragma unroll
        for (int k = 0; k < G; ++k)
            if (group_open(x[k], d, wmin))
                sh.group[__hip_atomic_fetch_add(&sh.listed, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)] =
                    (uint16_t)(lo.c + k * lo.L);
    __syncthreads();
}

// The keys of a sparse round's groups (sh.group) to their owners; ordered after
// the streaming by a workgroup barrier.
template <int T, int G, typename E>
__device__ __forceinline__ void take_sparse(Cols<G, E>& cs, const Layout& lo, uint32_t ng, SharedSolve<T>& sh) {
    if (lo.r != 0) return;
    key_t<E>* sp = reinterpret_cast<key_t<E>*>(sh.sparse);
    for (uint32_t i = 0; i < ng; ++i)
#pragma unroll
        for (int k = 0; k < G; ++k)
            if ((int)sh.group[i] == lo.c + k * lo.L)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    cs.best[k][j] = sp[4 * i + j];
                    sp[4 * i + j] = key_none<E>();
                }
}

struct SolveStats {
    unsigned long long rounds, settled, fallbacks, barriers;
    uint32_t status;
};

// The workgroup's LDS state, at namespace scope so that solver variants compiled
// as separate functions still address it as LDS.
template <int T>
__shared__ SharedSolve<T> g_sh;

// bit of local column v (0 <= v < width) if this thread owns it, else 0
__device__ __forceinline__ uint32_t owner_bit(const Layout& lo, int64_t v, int width) {
    if (v < 0 || v >= width || lo.r != 0) return 0;
    const int64_t gi = v >> 2;
    if (gi % lo.L != lo.c) return 0;
    const int k = (int)(gi / lo.L);
    return 1u << (4 * k + (int)(v & 3));
}

// ---------------------------------------------------------------------------
// What cannot change the result is not read.  A row of a bucket at d can lower
// only open vertices above d (above d + wmin, where a smallest weight is known:
// compact copies), so a round reads no row once there is none, and only the column
// groups that hold one when they are few against the rows (sparse_round).  (Masking
// the other lanes in every round was slower: n=1024, one workgroup, cold caches,
// 163 us against 155; the batches of rows, not their bytes, take the time.)  Where weights are small against
// the vertices' degrees the last buckets hold most vertices and few are left:
// n=65536, p=0.5, weights up to 1000 has 36152 of its 65536 rows in the last
// bucket or the last but one (2.53 ms reading every row, 1.17 so).  `every_row` (a
// solve that asks for one kernel by its flag: measurements of Algorithm 1's whole
// loop) reads every row whole; so does literal mode.
//
// ---------------------------------------------------------------------------
// One workgroup, whole row.
//
// A round settles the bucket, streams its rows (sh.list16), merges the row
// partitions, and finds the next minimum and its bucket in one go.  It is bound
// by that chain, not by bytes, so it has as few workgroup barriers as the data
// needs: one when the merge is complete, one when the next minimum is known,
// one when the next bucket is listed (in no particular order: a round's result
// is a minimum over its rows).  (Nine barriers and four block reductions before:
// n=256, p=0.1, 36 rounds, 97 us a call, now 70.)
// ---------------------------------------------------------------------------
template <int T, int G, int U, typename E>
__device__ __forceinline__ void solve_single(const E* __restrict__ W, int64_t ld, int32_t n, int32_t src,
                             int32_t* __restrict__ dist, int32_t* __restrict__ pred,
                             bool literal, bool every_row, uint32_t wmin, SharedSolve<T>& sh, SolveStats& st,
                             Ctl* trace) {
    every_row |= literal;
    const Layout lo = make_layout<T>(n);
    Cols<G, E> cs;
    init_cols(cs, lo, 0, n, src);
    clear_merge<T>(sh.mrg, 4 * T);
    if (threadIdx.x < 3) {
        sh.min3[threadIdx.x] = kNoKey;
        sh.count3[threadIdx.x] = 0;
        sh.open3[threadIdx.x] = 0;
    }
    if (threadIdx.x < 4 * kSparseGroups) sh.sparse[threadIdx.x] = kNoKey;
    if (threadIdx.x == 0) sh.listed = 0;
    if (threadIdx.x == 0) sh.list16[0] = (uint16_t)src;
    __syncthreads();
    uint32_t d = 0, u0 = (uint32_t)src, M = 1;
    bool redo = false;  // the round repeats the last one as one literal step (zero-weight hazard)
    uint32_t ng = ~0u;  // groups the round can lower
    uint32_t slot = 0;  // exchanges so far mod 3
    uint32_t neg = 0;
    uint32_t cand[G][4];
    for (;;) {
        const long long t_round = trace ? wall_clock64() : 0;
        const bool step = literal || redo;
        const uint32_t bucket = settle(cs, d, step, step ? owner_bit(lo, (int64_t)u0, n) : 0u);
        if (!step && sparse_round(ng, M, lo.P, ~0u)) {
            list_groups<T, G>(cs.x, d, wmin, lo, sh);
            for (uint32_t i = 0; i < ng; ++i)
                stream_sparse<T, E, false>(W, ld, 0, n, 4 * (int)sh.group[i], (int)M,
                                           [&](int e) { return (uint32_t)sh.list16[e]; },
                                           reinterpret_cast<key_t<E>*>(sh.sparse) + 4 * i);
            __syncthreads();
            if (threadIdx.x == 0) sh.listed = 0;
            take_sparse<T, G, E>(cs, lo, ng, sh);
        } else if (ng) {
            stream_rows<G, U, E>(cs, lo, W, ld, 0, n, sh.list16, (int)M);
            merge_partitions<T, G>(cs, lo, sh.mrg);
        }
        if (!redo) {
            ++st.rounds;
            if (trace && threadIdx.x == 0 && st.rounds <= (unsigned long long)kTraceCap) {
                trace->trace_t[st.rounds - 1] = t_round;
                trace->trace_m[st.rounds - 1] = M;
            }
        }
        // the would-be state and its lowest (dist, vertex)
        candidates(cs, d, ng != 0u, cand, neg);
        const bool owners = threadIdx.x < (unsigned)lo.L;  // whole waves, or the first lanes of wave 0
        if (threadIdx.x < (unsigned)max(lo.L, kWave)) {
            uint32_t dmin = 0xffffffffu;
#pragma unroll
            for (int k = 0; k < G; ++k)
#pragma unroll
                for (int j = 0; j < 4; ++j) dmin = min(dmin, cand[k][j]);
            dmin = wave_min32(dmin);
            uint32_t low = ~0u;
#pragma unroll
            for (int k = G - 1; k >= 0; --k)
#pragma unroll
                for (int j = 3; j >= 0; --j)
                    if (cand[k][j] == dmin) low = (uint32_t)local_col(lo, k, j);
            low = wave_min32(low);
            if (wave_lane() == 0)
                __hip_atomic_fetch_min(&sh.min3[slot], make_key(dmin, low), __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_WORKGROUP);
        }
        __syncthreads();
        const uint64_t key = sh.min3[slot];
        const uint32_t dn = scalar((uint32_t)(key >> 32));
        // the slot after the next one: its last readers passed the barrier before this one
        const uint32_t after = slot == 0 ? 2 : slot - 1;
        if (threadIdx.x == 0) {
            sh.min3[after] = kNoKey;
            sh.count3[after] = 0;
            sh.open3[after] = 0;
        }
        if (!step && dn == d) {
            // zero-weight hazard: discard the fused round and settle only u0, the
            // bucket's lowest vertex (one literal step)
            ++st.fallbacks;
            st.status |= kStatusZeroFallback;
            reopen(cs, bucket);
            reset_best(cs);
            redo = true;
            M = 1;
            if (threadIdx.x == 0) sh.list16[0] = (uint16_t)u0;
            __syncthreads();
            slot = slot == 2 ? 0 : slot + 1;
            continue;
        }
        redo = false;
        // a5/a6: relax
        if (lo.r == 0) commit(cs, cand);
        else reset_best(cs);
        st.settled += M;
        if (dn >= kInf) break;  // a4: nothing reachable is left
        d = dn;
        u0 = scalar((uint32_t)key);
        // a2/a3: the next bucket
        if (literal) {
            M = 1;
            if (threadIdx.x == 0) sh.list16[0] = (uint16_t)u0;
            __syncthreads();
        } else {
            if (owners) {
                if (!every_row) count_groups<T, G>(cs.x, d, wmin, slot, sh);
#pragma unroll
                for (int k = 0; k < G; ++k)
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const uint64_t at = wave_mask(cs.x[k][j] == d);
                        if (!at) continue;
                        uint32_t base = 0;
                        const int lead = __ffsll((unsigned long long)at) - 1;
                        if (wave_lane() == lead)
                            base = __hip_atomic_fetch_add(&sh.count3[slot], (uint32_t)__popcll(at), __ATOMIC_RELAXED,
                                                          __HIP_MEMORY_SCOPE_WORKGROUP);
                        base = lane_value(base, lead);
                        if (cs.x[k][j] == d) sh.list16[base + lanes_below(at)] = (uint16_t)local_col(lo, k, j);
                    }
            }
            __syncthreads();
            M = scalar(sh.count3[slot]);
            if (!every_row) {
                ng = scalar(sh.open3[slot]);
                if (ng == 0 && wmin == 0u) {
                    // the last bucket: its rows have nothing left to lower
                    ++st.rounds;
                    st.settled += M;
                    if (trace && threadIdx.x == 0 && st.rounds <= (unsigned long long)kTraceCap) {
                        trace->trace_t[st.rounds - 1] = wall_clock64();
                        trace->trace_m[st.rounds - 1] = M;
                    }
                    break;
                }
            }
        }
        slot = slot == 2 ? 0 : slot + 1;
    }
    if (neg & kSettled) st.status |= kStatusNegWeight;
    write_out(cs, lo, 0, n, dist, pred);  // a8
    if (trace && threadIdx.x == 0) {
        const unsigned long long nr = st.rounds < (unsigned long long)kTraceCap ? st.rounds : kTraceCap;
        trace->trace_t[nr] = wall_clock64();
        trace->trace_n = (uint32_t)nr;
    }
}
// ---------------------------------------------------------------------------
// Gang solve: `nwg` workgroups (ranks 0..nwg-1) each own a column slice of S
// columns and meet at one barrier per round.  Used by the whole-GPU kernel
// (the gang is the grid) and by the serving kernel (a gang per large query).
// ---------------------------------------------------------------------------

// Exchange number b of a gang of `members` workgroups, rank g: publishes this
// member's record in `slot` (filled before; records `stride` 64-bit words apart,
// the stamp in the first) and waits until every member's record there carries
// the same stamp.  Records and list entries are
// written and read with agent-scope atomic accesses (coherent across XCDs
// without cache writebacks or invalidates), so the only ordering needed is that
// a member's other stores are complete before its stamp: every wave waits for
// its stores (s_waitcnt 0) before the workgroup barrier, and thread 0 stores the
// stamp after it.  A reader reads a record's other fields only after seeing its
// stamp.  Thread t < members polls record t; nothing is counted in a shared
// word.  Gives up after `timeout` wall-clock ticks (returns false) so that a
// gang that is not co-resident cannot hang.  stamp = exchange_stamp(epoch, b)
// with an epoch unique to this use of the records' memory, so neither a record
// nor any other word left there by an earlier use ever matches.
template <int T>
__device__ __forceinline__ bool stamp_exchange(uint64_t* slot, size_t stride, int g, uint64_t stamp,
                                               uint32_t members, long long timeout, Red<T>& red) {
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if (members == 1) return true;  // one workgroup: its own barrier orders everything
    if (threadIdx.x == 0) {
        stress_delay((uint32_t)(stamp ^ (stamp >> 29)));
        __builtin_amdgcn_s_waitcnt(0);
        st_agent(&slot[(size_t)g * stride], stamp);
    }
    int late = 0;
    if (threadIdx.x < members) {
        // polls back off (up to ~1 us apart) so that members waiting through a
        // long round do not load the memory system the others are streaming from
        const long long t0 = wall_clock64();
        unsigned naps = 1;
        while (ld_agent(&slot[(size_t)threadIdx.x * stride]) != stamp) {
            for (unsigned i = 0; i < naps; ++i) __builtin_amdgcn_s_sleep(1);
            if (naps < 32) naps <<= 1;
            if (wall_clock64() - t0 > timeout) {
                late = 1;
                break;
            }
        }
    }
    return !block_any<T>(late, red);
}

// The exchange over 32-byte Pub records (stamp first).
template <int T>
__device__ __forceinline__ bool gang_exchange(Pub* slot, int g, uint64_t stamp, uint32_t members, long long timeout,
                                              Red<T>& red) {
    return stamp_exchange<T>(&slot->stamp, sizeof(Pub) / sizeof(uint64_t), g, stamp, members, timeout, red);
}

// Thread 0 of each member calls this once when it is done with the gang's
// words; the last of `members` resets them for the next use.  Returns true in
// the last member.
__device__ __forceinline__ bool gang_leave(Bar* bw, uint32_t members) {
    stress_delay(0xfffffffeu);
    const uint32_t prev = __hip_atomic_fetch_add(&bw->exit, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
    if (prev != members - 1) return false;
    __hip_atomic_store(&bw->bar, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(&bw->gen, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(&bw->exit, 0u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
    return true;
}

// Members of a gang come together (a batched launch, before they solve).  Each counts
// itself in *word (0 before).  Other work, on other streams, can keep some of a gang's
// workgroups from starting for as long as it runs, and itself wait for the compute
// units that the others hold; so the first part, whose ticket comes before the others',
// gives up after `limit`: it marks the gang broken and solves the item alone, and a
// member that finds the mark leaves.  True: all `members` are here, each on the GPU.
// (One thread of each member calls it; a member's own wait ends because part 0, which
// runs when any of them does, either sees them all or breaks the gang.)
constexpr uint32_t kGangBroken = 0x80000000u;
template <class Now, class Pause>
__host__ __device__ inline bool gang_meet(uint32_t* word, int32_t part, uint32_t members, long long limit, Now now,
                                          Pause pause) {
    uint32_t v = __hip_atomic_fetch_add(word, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1u;
    const long long t0 = now();
    while (v < members) {  // a mark makes it larger
        if (part == 0 && now() - t0 >= limit) {
            if (__hip_atomic_compare_exchange_strong(word, &v, v | kGangBroken, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                     __HIP_MEMORY_SCOPE_AGENT))
                return false;
            continue;
        }
        pause();
        v = __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    return (v & kGangBroken) == 0;
}

// The last workgroup of a launch publishes the launch's statistics and resets
// the barrier words, the ticket counter and the accumulators for the next launch.
__device__ __forceinline__ void finish_launch(Ctl* ctl, const SolveStats& st, bool add_stats) {
    if (threadIdx.x != 0) return;
    if (st.status) __hip_atomic_fetch_or(&ctl->status_acc, st.status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (add_stats) {
        __hip_atomic_fetch_add(&ctl->acc[kStatRounds], st.rounds, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_fetch_add(&ctl->acc[kStatSettled], st.settled, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_fetch_add(&ctl->acc[kStatFallbacks], st.fallbacks, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_fetch_add(&ctl->acc[kStatBarriers], st.barriers, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    stress_delay(0xffffffffu);
    const uint32_t prev = __hip_atomic_fetch_add(&ctl->b.exit, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
    if (prev == gridDim.x - 1) {
        for (int i = 0; i < kStatCount; ++i) {
            ctl->last[i] = __hip_atomic_load(&ctl->acc[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(&ctl->acc[i], 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        ctl->status = __hip_atomic_exchange(&ctl->status_acc, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        // a new epoch for the next launch's exchange records
        __hip_atomic_fetch_add(&ctl->epoch, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(&ctl->next_item, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(&ctl->b.bar, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(&ctl->b.gen, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(&ctl->b.exit, 0u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
    }
}

// Clear this member's tagged words (both slots of its record and of its list
// region) before the solve's first exchange; see tag_word.
template <int T>
__device__ __forceinline__ void clear_tagged(uint64_t* __restrict__ recs, uint64_t* __restrict__ lists,
                                             uint32_t* __restrict__ ctr, uint64_t* __restrict__ done, int g, int nwg,
                                             int S) {
    if (threadIdx.x < 2 * kRecFields)
        st_agent(rec_word(recs, nwg, threadIdx.x / kRecFields, threadIdx.x % kRecFields, g), (uint64_t)0);
    if (threadIdx.x == 2 * kRecFields) st_agent(&done[2 * g], (uint64_t)0);
    if (threadIdx.x == 2 * kRecFields + 1) st_agent(&ctr[4 * g], 0u);
    if (threadIdx.x == 2 * kRecFields + 2) st_agent(&ctr[4 * g + 1], 0u);
    for (int i = threadIdx.x; i < 2 * S; i += T) {
        const int s = i >= S ? 1 : 0;
        st_agent(&lists[((size_t)s * nwg + g) * S + (i - s * S)], (uint64_t)0);
    }
}

// Publish this workgroup's record for exchange `tag`: the lowest (dist, vertex)
// key among `cand` (one would-be dist per owned column; 0x80000000 and above =
// settled or no column), the vertices of the slice at that dist (list entries;
// none if `entries` is false) and, for a fused round of dist d, the zero-weight
// hazard flag (a candidate still at d, see candidates), every word tagged.
// Nothing waits for the stores: readers check each word's tag.
template <int T, int G, bool NARROW>
__device__ __forceinline__ void publish(const uint32_t (&cand)[G][4], const Layout& lo, int64_t col0, uint32_t d,
                                        bool fused, bool entries, uint32_t tag, uint64_t* __restrict__ recs, int nwg,
                                        int g, uint64_t* __restrict__ list, SharedSolve<T>& sh) {
    uint64_t* rec = rec_word(recs, nwg, (tag - 1) & 1, 0, g);
    if (NARROW || (G == 1 && lo.L <= kWave)) {
        // the owners are lanes of wave 0, 4 ascending columns each: one 32-bit
        // minimum, the rest from ballots
        if (threadIdx.x >= kWave) return;
        const uint32_t dmin = wave_min32(min(min(cand[0][0], cand[0][1]), min(cand[0][2], cand[0][3])));
        uint64_t at[4];
        uint32_t total = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            at[j] = wave_mask(cand[0][j] == dmin);  // of no interest when dmin >= kInf: the solve ends
            total += (uint32_t)__popcll(at[j]);
        }
        // the lane of the lowest vertex stores the record
        if (wave_lane() == (int)__builtin_ctzll(at[0] | at[1] | at[2] | at[3])) {
            stress_delay(2u * tag);
            const int j = cand[0][0] == dmin ? 0 : cand[0][1] == dmin ? 1 : cand[0][2] == dmin ? 2 : 3;
            st_agent(&rec[kRecRest], rec_rest(tag, (uint32_t)(col0 + local_col(lo, 0, j)), total,
                                              fused && dmin == d ? 1u : 0u));
            st_agent(&rec[kRecDist], tag_word(tag, dmin));
        }
        if (entries) {
            stress_delay(2u * tag + 1u);
            uint32_t rank = 0;
#pragma unroll
            for (int j = 0; j < 4; ++j) rank += lanes_below(at[j]);
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (cand[0][j] == dmin)
                    st_agent(&list[rank++], tag_word(tag, (uint32_t)(col0 + local_col(lo, 0, j))));
        }
        return;
    }
    if (NARROW) return;
    // the owners are whole waves: each finds its minimum, two workgroup barriers tell the
    // slice's and the entries before each wave's (sh.min3[0] is all ones before: thread 0
    // sets it back before the barrier of the exchange)
    const bool owners = threadIdx.x < (unsigned)lo.L;
    if (owners) {
        uint32_t dmin = 0xffffffffu;
#pragma unroll
        for (int k = 0; k < G; ++k)
#pragma unroll
            for (int j = 0; j < 4; ++j) dmin = min(dmin, cand[k][j]);
        dmin = wave_min32(dmin);
        uint32_t low = ~0u;
#pragma unroll
        for (int k = G - 1; k >= 0; --k)
#pragma unroll
            for (int j = 3; j >= 0; --j)
                if (cand[k][j] == dmin) low = (uint32_t)local_col(lo, k, j);
        low = wave_min32(low);
        if (wave_lane() == 0)
            __hip_atomic_fetch_min(&sh.min3[0], make_key(dmin, low), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
    __syncthreads();
    const uint64_t key = sh.min3[0];
    const uint32_t dmin = scalar((uint32_t)(key >> 32));
    uint32_t mask = 0, inc = 0;
    if (owners) {
        if (dmin < kInf) {
#pragma unroll
            for (int k = 0; k < G; ++k)
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (cand[k][j] == dmin) mask |= 1u << (4 * k + j);
        }
        inc = wave_prefix32((uint32_t)__popc(mask));
        if (wave_lane() == kWave - 1) sh.red.b[threadIdx.x / kWave] = inc;
    }
    __syncthreads();
    const int w = threadIdx.x / kWave, waves = lo.L / kWave;
    uint32_t total = 0, before = 0;
    if (owners) {
        for (int i = 0; i < waves; ++i) {
            const uint32_t c = sh.red.b[i];
            before += i < w ? c : 0u;
            total += c;
        }
    }
    if (entries && mask) {
        stress_delay(2u * tag + 1u);
        uint32_t rank = before + inc - (uint32_t)__popc(mask);
#pragma unroll
        for (int k = 0; k < G; ++k)
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (mask >> (4 * k + j) & 1u)
                    st_agent(&list[rank++], tag_word(tag, (uint32_t)(col0 + local_col(lo, k, j))));
    }
    if (threadIdx.x == 0) {
        stress_delay(2u * tag);
        st_agent(&rec[kRecRest], rec_rest(tag, (uint32_t)col0 + (uint32_t)key, total, fused && dmin == d ? 1u : 0u));
        st_agent(&rec[kRecDist], tag_word(tag, dmin));
        sh.min3[0] = kNoKey;
    }
}

// Bounded wait for a tagged word: returns it once it carries `tag`; on time-out
// sets `late` and returns the last value read.
__device__ __forceinline__ uint64_t wait_tag(const uint64_t* p, uint64_t w, uint32_t tag, long long timeout,
                                             uint32_t& late) {
    if (word_tag(w) == tag) return w;
    const long long t0 = wall_clock64();
    for (;;) {
        __builtin_amdgcn_s_sleep(1);
        w = ld_agent(p);
        if (word_tag(w) == tag) return w;
        if (wall_clock64() - t0 > timeout) {
            late = 1;
            return w;
        }
    }
}

// The wave's part of read_records: lane l polls members l + 64 k, k < KM, and the
// wave leaves the exchange's result in sh.res[tag & 1] and the bucket in sh.list (staged)
// or its counts and offsets in sh.cnt / sh.pre.
template <int T, int G, bool NARROW, int KM>
__device__ __forceinline__ void read_wave(uint64_t* recs, const uint64_t* __restrict__ rl, int S, int nwg,
                                          uint32_t wmin, uint32_t tag, long long timeout, SharedSolve<T>& sh, const Pub* stamps,
                                          uint64_t stamp, const uint32_t (&cand)[G][4]) {
    const int l = wave_lane();  // not threadIdx.x: addresses hoisted out of the round loop would spill
    uint32_t late = sh.stage_late;
    // Every poll issues all of its loads before it checks any (member indexes
    // clamped to the last member): a load per branch would be waited for before
    // the next one, KM round trips per poll instead of one.  Polls back off (up to
    // ~0.1 us apart) so that members waiting through a long round do not load the
    // memory system the others are streaming from.  The clock is read from the
    // first poll that misses a record on; a limit of 0 ends that poll.
    long long t0 = 0;
    unsigned naps = 0;
    auto give_up = [&]() {
        const long long now = wall_clock64();
        if (t0 == 0) t0 = now;
        if (now - t0 >= timeout) return true;
        for (unsigned i = 0; i < naps; ++i) __builtin_amdgcn_s_sleep(1);
        naps = naps ? (naps < 4 ? naps << 1 : naps) : 1;
        return false;
    };
    if (stamps) {
        for (;;) {
            uint64_t sv[KM];
#pragma unroll
            for (int k = 0; k < KM; ++k) sv[k] = ld_agent(&stamps[min(l + kWave * k, nwg - 1)].stamp);
            bool there = true;
#pragma unroll
            for (int k = 0; k < KM; ++k) there = there && sv[k] == stamp;
            if (!wave_mask(!there)) break;
            if (give_up()) {
                late = 1;
                break;
            }
        }
    }
    const uint32_t rtag = tag & kRestTagMask;
    uint64_t a[KM], r[KM];
    for (;;) {
#pragma unroll
        for (int k = 0; k < KM; ++k) {
            const uint64_t* w = rec_word(recs, nwg, (tag - 1) & 1, 0, min(l + kWave * k, nwg - 1));
            a[k] = ld_agent(&w[kRecDist]);
            r[k] = ld_agent(&w[kRecRest]);
        }
        bool there = true;
#pragma unroll
        for (int k = 0; k < KM; ++k) there = there && word_tag(a[k]) == tag && rest_tag(r[k]) == rtag;
        if (!wave_mask(!there) || late) break;
        if (give_up()) {
            late = 1;
            break;
        }
    }
    late = wave_mask(late != 0) ? 1u : 0u;
    uint32_t dist[KM], least = 0xffffffffu;
#pragma unroll
    for (int k = 0; k < KM; ++k) {
        dist[k] = l + kWave * k < nwg ? (uint32_t)a[k] : 0xffffffffu;
        least = min(least, dist[k]);
    }
    const uint32_t d = wave_min32(least);
    // Members own ascending columns, so the bucket's lowest vertex is that of its
    // lowest member.  The bucket is the concatenation of the bucket records' lists
    // in position order, position 4 l + k holding member l + 64 k (entry_addr).
    uint32_t low = 0, hazard = 0, local = 0, most = 0;
    uint32_t c[KM];
#pragma unroll
    for (int k = KM - 1; k >= 0; --k) {
        const uint64_t at = wave_mask(dist[k] == d);
        if (at) low = lane_value(rest_vertex(r[k]), (int)__builtin_ctzll(at));
        hazard |= rest_zero(r[k]);
        c[k] = dist[k] == d ? rest_count(r[k]) : 0u;
        local += c[k];
        most = max(most, c[k]);
    }
    const uint32_t inc = wave_prefix32(local);
    uint32_t run = inc - local;
    const bool small = rl && !late && wave_mask(most > (G == 1 ? 2u : 1u)) == 0;
    if (small) {
        // at most 2 x 256 entries: they fit the staging list
        if (G == 1 && wave_mask(most > 1u)) {
            uint64_t w[KM];
#pragma unroll
            for (int k = 0; k < KM; ++k) w[k] = c[k] > 1u ? ld_agent(&rl[(uint32_t)(l + kWave * k) * (uint32_t)S + 1]) : 0;
            uint32_t pos = run;
#pragma unroll
            for (int k = 0; k < KM; ++k) {
                if (c[k] > 1u) {
                    uint32_t miss = 0;
                    const uint64_t e =
                        wait_tag(&rl[(uint32_t)(l + kWave * k) * (uint32_t)S + 1], w[k], tag, timeout, miss);
                    // a time-out stages a valid row; the solve then ends with the time-out status
                    sh.list[pos + 1] = (int32_t)(miss ? rest_vertex(r[k]) : (uint32_t)e);
                    if (miss) sh.stage_late = 1u;
                }
                pos += c[k];
            }
        }
#pragma unroll
        for (int k = 0; k < KM; ++k) {
            if (c[k]) sh.list[run] = (int32_t)rest_vertex(r[k]);
            run += c[k];
        }
    } else {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            sh.pre[4 * l + k] = run;
            sh.cnt[4 * l + k] = k < KM ? c[k < KM ? k : 0] : 0u;
            if (k < KM) run += c[k < KM ? k : 0];
        }
    }
    hazard = wave_mask(hazard != 0) ? 1u : 0u;
    // the slice's owners are lanes of this wave: their groups the next round reads
    const uint64_t open = NARROW ? wave_mask(group_open(cand[0], d, wmin)) : 0ull;
    if (l == kWave - 1) {  // one 16-byte store here, one load in every thread
        auto& res = sh.res[tag & 1u];
        res.d = d;
        res.vert = low;
        res.rows = inc;
        res.flags = hazard | (small ? 2u : 0u) | (late << 2);
        if (NARROW) sh.res_need[tag & 1u] = open;
    }
}

// Exchange `tag` from the reader's side: waits for the gang's nwg tagged records
// of its slot and reduces them.  `stamps` (the solve's first exchange only):
// each member's tagged words are read only after its stamp, which it stored
// once its cleared words were in place, has been seen (in an earlier poll, so
// the tagged loads are issued after the stamp load returned).
// d_out, u_out = the lowest key's dist and vertex, Z = the OR of the hazard
// flags; for the round's bucket (records whose key has dist d) each record's count and offset go to
// sh.cnt / sh.pre and their sum to M.  Wave 0 polls and reduces (lane l takes
// members l, l + 64, l + 128, l + 192) and shares the results through LDS after
// one workgroup barrier; gangs of more than 256 members take a block-wide path.
// `rl` (null: no entries wanted): the gang's lists of this exchange.  When no
// member has more than two bucket vertices (one, where a thread holds several
// column groups and the list's order is not the vertices') the wave stages the
// whole bucket in sh.list itself, the first entry of each member from its
// record, and *staged tells: small rounds are bound by their chain of memory
// and LDS round trips, and this takes the entry lookup, its load and one barrier
// off it.  (Bare kernel, 64 workgroups, n=4096, p=0.002, 962 rounds: 4.84 ms before the
// records' layout, the 32-bit reductions, the short batches and the staging, 2.92 ms
// with them; n=16384, p=0.01, 17 rounds: 305 and 265 us.)  Returns false if a member's record, or an entry of the last round's bucket
// (sh.stage_late), did not arrive within `timeout` ticks.
template <int T, int G, bool NARROW>
__device__ __forceinline__ bool read_records(uint64_t* recs, const uint64_t* __restrict__ rl, int S, int nwg,
                                             uint32_t wmin, uint32_t tag, long long timeout, SharedSolve<T>& sh,
                                             uint32_t& d_out,
                                             uint32_t& u_out, uint32_t& Z, uint32_t& M, bool& staged, uint64_t& open,
                                             const Pub* stamps, uint64_t stamp, const uint32_t (&cand)[G][4]) {
    staged = false;
    if (NARROW || nwg <= 4 * kWave) {
        if (threadIdx.x < kWave) {
            // members 64 to 255 of a gang of at most 64 do not exist
            if (nwg <= kWave) read_wave<T, G, NARROW, 1>(recs, rl, S, nwg, wmin, tag, timeout, sh, stamps, stamp, cand);
            else read_wave<T, G, NARROW, 4>(recs, rl, S, nwg, wmin, tag, timeout, sh, stamps, stamp, cand);
        }
        __syncthreads();
        stress_wave_delay(tag);
        // the same in every thread: scalar registers
        const auto res = sh.res[tag & 1u];
        d_out = scalar(res.d);
        u_out = scalar(res.vert);
        M = scalar(res.rows);
        const uint32_t z = scalar(res.flags);
        Z = z & 1u;
        staged = (z & 2u) != 0;
        if (NARROW) {
            const uint64_t o = sh.res_need[tag & 1u];
            open = ((uint64_t)scalar((uint32_t)(o >> 32)) << 32) | scalar((uint32_t)o);
        }
        return (z & 4u) == 0;
    }
    const uint32_t slot = (tag - 1) & 1;
    const uint32_t rtag = tag & kRestTagMask;
    if (NARROW) return false;
    uint64_t key = kNoKey;
    uint32_t c = 0, f = 0, late = 0;
    if ((int)threadIdx.x < nwg) {
        const int m = (int)threadIdx.x;
        if (stamps) {
            const long long t0 = wall_clock64();
            while (ld_agent(&stamps[m].stamp) != stamp)
                if (wall_clock64() - t0 > timeout) {
                    late = 1;
                    break;
                }
        }
        const uint64_t* w = rec_word(recs, nwg, slot, 0, m);
        const uint64_t a = wait_tag(&w[kRecDist], ld_agent(&w[kRecDist]), tag, timeout, late);
        uint64_t r = ld_agent(&w[kRecRest]);
        const long long t1 = wall_clock64();
        while (rest_tag(r) != rtag) {
            if (wall_clock64() - t1 > timeout) {
                late = 1;
                break;
            }
            r = ld_agent(&w[kRecRest]);
        }
        key = make_key((uint32_t)a, rest_vertex(r));
        c = rest_count(r);
        f = rest_zero(r) | (late << 1);
    }
    if (threadIdx.x == 0 && sh.stage_late) f |= 2u;
    uint64_t K = key;
    Z = f;
    block_min_or<T>(K, Z, sh.red);
    d_out = (uint32_t)(K >> 32);
    u_out = (uint32_t)K;
    if (key == kNoKey || (uint32_t)(key >> 32) != d_out) c = 0;
    const uint32_t pre = block_excl_scan<T>(c, M, sh.red);
    if ((int)threadIdx.x < nwg) {
        sh.pre[threadIdx.x] = pre;
        sh.cnt[threadIdx.x] = c;
    }
    __syncthreads();
    const bool ok = (Z & 2u) == 0;
    Z &= 1u;
    return ok;
}

// Address of entry e of the round's bucket, the concatenation of the lists of
// the records whose minimum equals d.  sh.pre / sh.cnt hold each position's
// prefix offset and count; with at most 256 members (read_records' wave path)
// position 4 l + k holds member l + 64 k (positions of absent members count 0),
// otherwise position m holds member m.
template <int T>
__device__ __forceinline__ const uint64_t* entry_addr(const SharedSolve<T>& sh, const uint64_t* __restrict__ rl,
                                                      int nwg, int S, uint32_t e) {
    const bool packed = nwg <= 4 * kWave;
    int lo_i = 0, hi_i = packed ? 4 * kWave - 1 : nwg - 1;  // last position whose prefix is <= e
    while (lo_i < hi_i) {
        const int mid = (lo_i + hi_i + 1) >> 1;
        if (sh.pre[mid] <= e) lo_i = mid;
        else hi_i = mid - 1;
    }
    const int m = packed ? (lo_i & 3) * kWave + (lo_i >> 2) : lo_i;
    return &rl[(size_t)m * S + (e - sh.pre[lo_i])];
}

// Rank g of a gang of nwg workgroups.  gw: the gang's exchange memory (see
// gang_words_bytes).  Returns false if a wait timed out.  `trace` (may be null)
// receives rank 0's round trace.  b0: exchanges the gang's words have already
// counted in this use (a solve that follows another one on the same words
// continues the numbering); epoch: unique to this use of the words (stamps of
// the first exchange).
//
// BAL: pair balancing of large rounds.  Equal slices do not take equal time
// (workgroups on some XCDs stream measurably slower), and a round lasts as long
// as its slowest member.  In a round of at least kPairChunks chunks, members g
// and g ^ 1 claim the rows of their own slice from the front of a counter, a
// staging chunk (kCap rows) at a time; one that runs out claims the partner's
// remaining rows from the back, kPairUnit rows at a time, streams them over the
// partner's columns, then hands the partial minima over (partial keys, then a
// tagged done word once they are in memory).  The counter word counts units of
// kPairUnit rows, front claims in its low 16 bits and back claims in its high
// 16 bits; the atomic adds serialise the claims, a claim made when front +
// back < units is valid, a front claim stops at the back claims made before it,
// and later back claims see its whole increment, so no row is taken twice or
// left out.  Claims are made two ahead so that their latency hides behind the
// streaming; the helper's claims from the back do not wait for the rows the
// owner has reserved at the front.  Each member has two
// counters (round parity) and resets one only after reading the exchange that
// follows the round that used it, when both members' claims on it have
// returned, and before its next publish (the partner claims on it again only
// after that publish).
template <int T, int G, int U, typename E, bool NT = false, bool BAL = false, bool NARROW = false>
__device__ __forceinline__ bool solve_gang(const E* __restrict__ W, int64_t ld, int32_t n, int32_t src,
                           int32_t* __restrict__ dist, int32_t* __restrict__ pred, bool literal,
                           bool every_row, uint32_t wmin, int S, int g, int nwg, long long timeout, GangWords gw,
                           SharedSolve<T>& sh, SolveStats& st, Ctl* trace, uint32_t epoch, uint32_t b0 = 0) {
    static_assert(T == kCap, "one staged bucket entry per thread");
    static_assert(!BAL || sizeof(E) == 4, "pair balancing keeps 64-bit keys");
    static_assert(!NARROW || G == 1, "narrow slices have one column group per lane");
    if (sizeof(E) == 4) wmin = 0u;  // no smallest weight is known of the caller's matrix
    every_row |= literal;
    const int64_t col0 = (int64_t)g * S;
    const int width = (int)max((int64_t)0, min((int64_t)S, (int64_t)n - col0));
    const Layout lo = make_layout<T>(S);
    Cols<G, E> cs;
    init_cols(cs, lo, col0, width, src);
    clear_merge<T>(sh.mrg, 4 * T);
    // nwg * S words fit 32 bits: at most 1024 members of 16384 columns
    auto list_of = [&](uint32_t x, int m) { return gw.lists + (((x - 1) & 1u) * (uint32_t)nwg + (uint32_t)m) * (uint32_t)S; };

    uint32_t b = b0;  // exchanges passed
    bool ok = true;
    // Clear this member's tagged words, then stamp its record for the first
    // exchange (b0 + 1) once they are in place: readers take its tagged words
    // only after seeing that stamp (read_records).
    clear_tagged<T>(gw.recs, gw.lists, gw.ctr, gw.done, g, nwg, S);
    // pair balancing: the partner, counter slots that a round has used and not
    // yet reset, and the value of the last reset (used before the next publish)
    const int pg = g ^ 1;
    const bool paired = BAL && pg < nwg && lo.P > 1;
    uint32_t used = 0, reset_old = 0;
    // the same in every thread (it comes from a load): a scalar register
    const uint64_t stamp1 = exchange_stamp((uint32_t)__builtin_amdgcn_readfirstlane((int)epoch), b0 + 1);
    const Pub* stamps1 = gw.pubs + (size_t)(b0 & 1) * nwg;
    if (threadIdx.x == 0) sh.stage_late = 0u;
    if (threadIdx.x < 3) sh.open3[threadIdx.x] = 0u;
    if (threadIdx.x == 0) sh.min3[0] = kNoKey;
    if (threadIdx.x == 0) sh.listed = 0u;
    if (threadIdx.x < 4 * kSparseGroups) sh.sparse[threadIdx.x] = kNoKey;
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if (threadIdx.x == 0) {
        stress_delay((uint32_t)(stamp1 ^ (stamp1 >> 29)));
        __builtin_amdgcn_s_waitcnt(0);
        st_agent(&gw.pubs[(size_t)(b0 & 1) * nwg + g].stamp, stamp1);
    }
    // The first round's bucket, {src} at distance 0, is the same in every
    // member's view: no exchange precedes it.
    uint32_t d = 0, u0 = (uint32_t)src, M = 1;
    bool first = true;
    bool staged = false;  // the bucket is in sh.list already (read_records)
    // groups of the slice that the round can lower, and (narrow slices) the lanes that
    // own them
    uint32_t ng = ~0u, slot3 = 0;
    uint64_t open = ~0ull;
    bool redo = false;    // the round repeats the last one as one literal step (zero-weight hazard)
    uint32_t rounds = 0, settled = 0, fallbacks = 0, neg = 0;
    const bool tracer = trace && g == 0 && threadIdx.x == 0;
    uint32_t cand[G][4];
    for (;;) {
        if (!redo) ++rounds;
        const long long t_round = tracer ? wall_clock64() : 0;
        // a literal step's one row, or a bucket that read_records staged: in sh.list already
        const bool step = literal || redo;
        if (step) M = 1;
        const uint32_t bucket = settle(cs, d, step, step ? owner_bit(lo, (int64_t)u0 - col0, width) : 0u);
        if (step && threadIdx.x == 0) sh.list[0] = (int32_t)u0;
        const bool ready = step || staged;
        const uint64_t* rl = list_of(b, 0);
        // entry e of the bucket into sh.list[threadIdx.x]; w: its word as loaded
        auto stage = [&](uint32_t e, uint64_t w) {
            uint32_t late = 0;
            if (word_tag(w) != b) w = wait_tag(entry_addr<T>(sh, rl, nwg, S, e), w, b, timeout, late);
            // a time-out stages a valid row; the solve then ends with the time-out status
            sh.list[threadIdx.x] = late ? (int32_t)u0 : (int32_t)(uint32_t)w;
            if (late) sh.stage_late = 1u;
        };
        const uint32_t C = (M + kCap - 1) / kCap;
        // the whole-GPU kernels stream from memory at its rate; batched and served gangs do not
        const bool sparse = !step && sparse_round(ng, M, lo.P, NT ? (uint32_t)S * (uint32_t)sizeof(E) : ~0u);
        if (paired && C >= kPairChunks && (ng == 0 || sparse)) {
            // leave the partner none of this member's rows to claim
            used |= 1u << (b & 1);
            if (threadIdx.x == 0)
                __hip_atomic_fetch_add(&gw.ctr[4 * g + (b & 1)], (M + kPairUnit - 1) / kPairUnit, __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_AGENT);
        }
        if (ng == 0) {
            // nothing in this slice can be lowered
        } else if (sparse) {
            auto row = [&](int e) -> uint32_t {
                if (staged) return (uint32_t)sh.list[e];
                const uint64_t* a = entry_addr<T>(sh, rl, nwg, S, (uint32_t)e);
                uint32_t late = 0;
                const uint64_t w = wait_tag(a, ld_agent(a), b, timeout, late);
                if (late) sh.stage_late = 1u;
                return late ? u0 : (uint32_t)w;
            };
            key_t<E>* sp = reinterpret_cast<key_t<E>*>(sh.sparse);
            if (NARROW) {
                uint32_t i = 0;
                for (uint64_t o = open; o; o &= o - 1, ++i)
                    stream_sparse<T, E, NT>(W, ld, col0, width, 4 * (int)__builtin_ctzll(o), (int)M, row, sp + 4 * i);
            } else {
                list_groups<T, G>(cs.x, d, wmin, lo, sh);
                for (uint32_t i = 0; i < ng; ++i)
                    stream_sparse<T, E, NT>(W, ld, col0, width, 4 * (int)sh.group[i], (int)M, row, sp + 4 * i);
            }
            __syncthreads();
            if (NARROW) {
                if (threadIdx.x < kWave && (open >> threadIdx.x & 1ull)) {
                    const uint32_t i = lanes_below(open);
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        cs.best[0][j] = sp[4 * i + j];
                        sp[4 * i + j] = key_none<E>();
                    }
                }
            } else {
                if (threadIdx.x == 0) sh.listed = 0u;
                take_sparse<T, G, E>(cs, lo, ng, sh);
            }
        } else if (paired && C >= kPairChunks) {
            const uint32_t slot = b & 1;
            const uint32_t tag = b + 1;  // the exchange this round publishes
            key_t<E>* keep = reinterpret_cast<key_t<E>*>(sh.mrg + 2 * T);
            uint32_t own = 0;
            for (int side = 0; side < 2; ++side) {
                const int m = side ? pg : g;
                const int64_t c0 = (int64_t)m * S;
                const int wd = (int)max((int64_t)0, min((int64_t)S, (int64_t)n - c0));
                uint32_t* ctr = &gw.ctr[4 * m + slot];
                // claims count units of kPairUnit rows: the owner takes a staging
                // chunk (kCap rows) at a time from the front, the helper one unit at
                // a time from the back
                constexpr uint32_t kChunkUnits = (uint32_t)kCap / kPairUnit;
                const uint32_t units = (M + kPairUnit - 1) / kPairUnit;
                uint32_t left = units;  // units unclaimed when the last decoded claim was made
                // rows [begin, begin + count) of a claim of `n` units (the counter
                // before it in `old`); count 0 if it came too late.  A front claim stops
                // at the back claims made before it; later back claims see its whole
                // increment and stay clear.
                auto rows_of = [&](uint32_t old, uint32_t nu, uint32_t& begin) -> uint32_t {
                    const uint32_t f = old & 0xffffu, h = old >> 16;
                    begin = 0;
                    left = f + h >= units ? 0u : units - f - h;
                    if (!left) return 0u;
                    const uint32_t u0 = side ? units - 1 - h : f;
                    const uint32_t u1 = side ? u0 + 1 : min(f + nu, units - h);
                    begin = u0 * kPairUnit;
                    return min(u1 * kPairUnit, M) - begin;
                };
                // the owner claims whole staging chunks, single units once few are
                // left (so that it reserves little for the helper to wait behind);
                // the helper always claims single units
                auto units_next = [&]() { return side || left <= 3 * kChunkUnits ? 1u : kChunkUnits; };
                auto inc_of = [&](uint32_t nu) { return side ? 0x10000u : nu; };
                if (side == 1) {
                    // keep this member's candidates while it streams rows for the partner
                    merge_partitions<T, G>(cs, lo, sh.mrg);
                    if (lo.r == 0)
#pragma unroll
                        for (int j = 0; j < 4; ++j) keep[j * lo.L + lo.c] = cs.best[0][j];
                    reset_best(cs);
                }
                const uint32_t nu0 = units_next();
                if (threadIdx.x == 0) {
                    if (side == 0) stress_delay(4u * tag + 3u);  // late starters: partners steal
                    sh.claim[0] = __hip_atomic_fetch_add(ctr, inc_of(nu0), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    sh.claim[1] = __hip_atomic_fetch_add(ctr, inc_of(nu0), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
                __syncthreads();
                uint32_t kb = 0, nb = 0;
                uint32_t kcnt = rows_of((uint32_t)__builtin_amdgcn_readfirstlane((int)sh.claim[0]), nu0, kb);
                uint32_t ncnt = rows_of((uint32_t)__builtin_amdgcn_readfirstlane((int)sh.claim[1]), nu0, nb);
                uint32_t chunks = 0;  // rows streamed on this side
                uint64_t w = 0;
                if (threadIdx.x < kcnt) w = ld_agent(entry_addr<T>(sh, rl, nwg, S, kb + threadIdx.x));
                while (kcnt) {
                    if (threadIdx.x < kcnt) stage(kb + threadIdx.x, w);
                    __syncthreads();
                    uint32_t a = 0xffffffffu;  // no further claim: nothing is left after the next one
                    const uint32_t nua = units_next();
                    if (ncnt) {
                        if (threadIdx.x < ncnt) w = ld_agent(entry_addr<T>(sh, rl, nwg, S, nb + threadIdx.x));
                        if (threadIdx.x == 0)
                            a = __hip_atomic_fetch_add(ctr, inc_of(nua), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    }
                    stream_rows<G, U, E, NT>(cs, lo, W, ld, c0, wd, sh.list, (int)kcnt);
                    if (threadIdx.x == 0) sh.claim[0] = a;
                    __syncthreads();
                    chunks += kcnt;
                    kb = nb;
                    kcnt = ncnt;
                    ncnt = rows_of((uint32_t)__builtin_amdgcn_readfirstlane((int)sh.claim[0]), nua, nb);
                }
                if (side == 0) {
                    own = chunks;
                    continue;
                }
                if (chunks) {
                    // the partner's share of its own columns: partial minima, then the
                    // tagged done word once they are in memory
                    merge_partitions<T, G>(cs, lo, sh.mrg);
                    if (lo.r == 0)
#pragma unroll
                        for (int j = 0; j < 4; ++j)
                            st_agent(&gw.part[(size_t)pg * S + 4 * lo.c + j], (uint64_t)cs.best[0][j]);
                    __builtin_amdgcn_s_waitcnt(0);
                    __syncthreads();
                    if (threadIdx.x == 0) st_agent(&gw.done[2 * pg], tag_word(tag, chunks));
                }
                // back to this member's own candidates
                if (lo.r == 0) {
#pragma unroll
                    for (int j = 0; j < 4; ++j) cs.best[0][j] = keep[j * lo.L + lo.c];
                } else {
                    reset_best(cs);
                }
            }
            if (own < M && lo.r == 0) {
                // the partner streamed the rest of this member's chunks: its partial minima
                uint32_t late = 0;
                (void)wait_tag(&gw.done[2 * g], ld_agent(&gw.done[2 * g]), tag, timeout, late);
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    cs.best[0][j] = key_min(cs.best[0][j], (key_t<E>)ld_agent(&gw.part[(size_t)g * S + 4 * lo.c + j]));
                if (late) sh.stage_late = 1u;
            }
            used |= 1u << slot;
        } else {
            // stage the bucket chunk by chunk; the next chunk's entries are loaded
            // while the current chunk's rows stream (the first round's one entry,
            // the source, is not loaded)
            uint64_t nxt = first ? tag_word(b, u0)
                         : !ready && threadIdx.x < M ? ld_agent(entry_addr<T>(sh, rl, nwg, S, threadIdx.x)) : 0;
            for (uint32_t e0 = 0; e0 < M; e0 += kCap) {
                const uint32_t e = e0 + threadIdx.x;
                if (!ready && e < M) stage(e, nxt);
                if (!staged || step) __syncthreads();  // a staged bucket: read_records ended with a barrier
                if (e + kCap < M) nxt = ld_agent(entry_addr<T>(sh, rl, nwg, S, e + kCap));
                stream_rows<G, U, E, NT>(cs, lo, W, ld, col0, width, sh.list,
                                         (int)min((uint32_t)kCap, M - e0));
                __syncthreads();
            }
        }
        // a single row went to partition 0, whose threads own the columns
        if (M > 1 && ng && !sparse) merge_partitions<T, G>(cs, lo, sh.mrg);
        if (tracer && !redo && rounds <= (uint32_t)kTraceCap) {
            trace->trace_t[rounds - 1] = t_round;
            trace->trace_m[rounds - 1] = M;
        }

        // would-be state if this round is applied (threads that own no column have
        // x = 0xffffffff, so theirs is no candidate)
        candidates(cs, d, ng != 0u, cand, neg);
        ++b;
        if (BAL) asm volatile("" ::"v"(reset_old));  // a counter reset has completed before this publish
        publish<T, G, NARROW>(cand, lo, col0, d, !step, !literal, b, gw.recs, nwg, g, list_of(b, g), sh);
        uint32_t Z, M_rec, d_next, u_next;
        uint64_t open_next = 0;
        ok = read_records<T, G, NARROW>(gw.recs, literal ? nullptr : list_of(b, 0), S, nwg, wmin, b, timeout, sh, d_next,
                                        u_next, Z, M_rec, staged, open_next, first ? stamps1 : nullptr, stamp1, cand);
        first = false;
        if (!ok) break;
        if (BAL && (used >> ((b - 1) & 1) & 1u)) {
            // every claim on the counter slot of the round just published has returned
            if (threadIdx.x == 0)
                reset_old = __hip_atomic_exchange(&gw.ctr[4 * g + ((b - 1) & 1)], 0u, __ATOMIC_RELAXED,
                                                  __HIP_MEMORY_SCOPE_AGENT);
            used &= ~(1u << ((b - 1) & 1));
        }
        if (Z) {
            // the fused round read a zero-weight edge out of its bucket: discard it
            // and settle only the bucket's lowest-index vertex (one literal step)
            ++fallbacks;
            st.status |= kStatusZeroFallback;
            reopen(cs, bucket);
            reset_best(cs);
            redo = true;
            continue;
        }
        redo = false;
        if (lo.r == 0) commit(cs, cand);
        else reset_best(cs);
        settled += M;
        d = d_next;
        if (d >= kInf) break;
        u0 = u_next;
        M = M_rec;
        if (!every_row) {
            if (NARROW) {
                open = open_next;
                ng = (uint32_t)__popcll(open);
            } else if (8u * (uint64_t)((uint32_t)n - settled - M) < (uint32_t)n) {
                // counted through LDS; not worth the barrier while an eighth of the
                // vertices is open beyond the bucket
                const uint32_t after = slot3 == 2 ? 0 : slot3 + 1;
                if (threadIdx.x == 0) sh.open3[after] = 0u;
                if (threadIdx.x < (unsigned)lo.L) count_groups<T, G>(cs.x, d, wmin, slot3, sh);
                __syncthreads();
                ng = scalar(sh.open3[slot3]);
                slot3 = after;
            } else {
                ng = ~0u;
            }
        }
    }
    st.rounds += rounds;
    st.settled += settled;
    st.fallbacks += fallbacks;
    if (neg & kSettled) st.status |= kStatusNegWeight;
    if (!ok) st.status |= kStatusTimeout;
    write_out(cs, lo, col0, width, dist, pred);
    st.barriers += b;
    if (tracer) {
        const uint32_t nr = min(rounds, (uint32_t)kTraceCap);
        trace->trace_t[nr] = wall_clock64();
        trace->trace_n = nr;
    }
    uint32_t s = st.status;
    uint64_t dummy = kNoKey;
    block_min_or<T>(dummy, s, sh.red);
    st.status = s;
    return ok;
}

}  // namespace sssp
