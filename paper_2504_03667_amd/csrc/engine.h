// Device engine shared by the dense-matrix Dijkstra kernels (gfx950, wave64).
//
// Vocabulary follows Algorithm 1 of the paper (Section III-A): dist[], pred[],
// visited[], the argmin vertex u, its distance d, and row u of the weight
// matrix W relaxed into dist/pred.
//
// A workgroup owns a contiguous slice of S columns (vertices) of the matrix —
// the single-GPU form of the paper's 1-D column division (Section III-B): it
// keeps dist[], pred[] and visited[] (the top bit of a settled dist, see Cols) of
// those vertices in registers and writes dist and pred out at the end, so every column has exactly one writer and no
// atomics are needed on dist or pred.
//
// Thread layout inside a workgroup of T threads.  The slice is cut into
// NG = ceil(S/4) column groups of 4 (one 128-bit load each).  L lanes cover the
// groups of one row (lane c owns groups c, c+L, ..., G of them), and the
// T/L = P row partitions stream different rows of the current bucket at the
// same time; partition 0 holds the slice state ("owner" threads).  After a
// round the P partial minima are merged through LDS into the owners.
//
// Per-column candidate of a round: the lexicographic minimum, over the rows u
// streamed, of the packed key (W[u][v] << 32 | u) compared as uint64.  Every
// row of one round has the same dist d, so this equals the minimum of
// (d + W[u][v], u): the lowest-index u wins a tie, which is what the strict
// '<' of Algorithm 1 yields when equal-distance rows are relaxed in index
// order.  Weights are read as uint32; INT32_MAX (no edge) then never improves
// anything, because d + INT32_MAX >= INT32_MAX >= dist[v].
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace sssp {

constexpr uint32_t kInf = 0x7fffffffu;
constexpr uint64_t kNoKey = ~0ull;
constexpr int kWave = 64;

// status bits (Ctl::status)
constexpr uint32_t kStatusTimeout = 1u;       // a grid barrier wait gave up
constexpr uint32_t kStatusNegWeight = 2u;     // a negative weight was the best candidate of a column
constexpr uint32_t kStatusZeroFallback = 4u;  // a zero-weight edge forced single-vertex steps

// statistics slots (Ctl::acc / Ctl::last)
enum { kStatRounds = 0, kStatSettled = 1, kStatFallbacks = 2, kStatBarriers = 3, kStatCount = 4 };

constexpr int kTraceCap = 256;  // rounds recorded per launch (round start time, bucket size)

// Barrier words of one group of workgroups (the whole grid, or a gang of a
// served query).  The arrival counter, the release word that waiters poll and
// the exit counter sit on separate 128-byte lines so that polling does not
// contend with arrivals.  All zero between uses: the last member to leave
// resets them.
struct Bar {
    uint32_t bar;  // arrivals
    uint32_t pad0[31];
    uint32_t gen;  // number of the last completed barrier
    uint32_t pad1[31];
    uint32_t exit;  // members that have left
    uint32_t pad2[31];
};

// Per-launch control block in device memory.  Zeroed once when allocated;
// every launch leaves it ready for the next (the last workgroup to finish
// resets the barrier words and moves the accumulators into `last`).
struct Ctl {
    Bar b;
    uint32_t status_acc;  // status bits OR-ed during the current launch
    uint32_t status;      // status of the last finished launch
    uint32_t trace_n;     // rounds recorded in trace_t / trace_m by the last launch
    uint32_t epoch;       // launches finished; stamps the exchange records of the next one
    unsigned long long acc[kStatCount];
    unsigned long long last[kStatCount];
    unsigned long long next_item;  // work-queue ticket counter (batched kernels)
    long long trace_t[kTraceCap + 1];  // wall-clock ticks at the start of each round, then the end
    uint32_t trace_m[kTraceCap];       // rows streamed in each round
};

// Stamp of exchange number b during use `epoch` of a gang's record memory.
// Bit 63 is always set, and nothing else ever stored in record or list memory
// has it: list entries are vertex indices below 2^31 (two per 64-bit word) or
// tagged words that keep it clear (tag_word, rec_rest, lc_word), and a record's key (which
// can be all ones) sits 8 bytes into its 32-byte record, while records always
// start at 32-byte offsets of the memory they share with earlier uses.  So a
// word left in the same memory by an earlier query or launch can never pass
// for the stamp a member is waiting for.
__host__ __device__ constexpr uint64_t exchange_stamp(uint32_t epoch, uint32_t b) {
    return (1ull << 63) | ((uint64_t)(epoch & 0x7fffffffu) << 32) | b;
}

// One workgroup's contribution to a round.  Written and read only with
// agent-scope atomic accesses, which are coherent across XCDs without cache
// writebacks or invalidates; `stamp` is stored last and tells the readers that
// the rest (and the workgroup's list entries) is in place.
struct alignas(32) Pub {
    uint64_t stamp;  // exchange_stamp(epoch, barrier number of the exchange it belongs to)
    uint64_t key;    // (would-be local min dist << 32) | lowest vertex at that dist; kNoKey if none
    uint32_t count;  // vertices of the slice at that dist, listed in the slot's list region
    uint32_t flags;  // bit 0: a zero-weight edge from the bucket to an unvisited vertex was seen
    uint64_t pad;
};
static_assert(sizeof(Pub) == 32, "stamped records are 32 bytes");

// Tagged exchange words.  After the first exchange of a gang's solve, every
// word a member publishes carries the number b of its exchange in the high 32
// bits (the word's tag) and a 32-bit value in the low ones, so a reader takes
// each word as soon as it shows the tag it waits for: a member neither waits
// for its own stores to complete nor orders them behind a stamp.  Each member
// clears its tagged words (tag 0) before the solve's first exchange, which
// uses stamps and so completes every member's earlier stores before anyone
// passes it; from then on a tagged word holds 0, a tag of an earlier exchange
// of the same solve (b - 2, b - 4, ... in the same slot) or the awaited one,
// and the tag of exchange b is b >= 1, below 2^32 because a solve of n < 2^31
// vertices has at most 2n + 1 exchanges.
__host__ __device__ constexpr uint64_t tag_word(uint32_t tag, uint32_t value) {
    return ((uint64_t)tag << 32) | value;
}
__host__ __device__ constexpr uint32_t word_tag(uint64_t w) { return (uint32_t)(w >> 32); }

// A gang's tagged records of the Dijkstra rounds: 64 bytes per member, its
// record of exchange parity 0 in the first half and of parity 1 in the second,
// so that no two members ever store into the same 64-byte line.  (Packed side by
// side, 16 members' stores share a line whose ownership moves between the XCDs:
// an exchange of 256 members with three packed words each took 2.7 us in a
// loop of bare exchanges, two words in a line of their own 1.7 us; 64 members
// 1.9 and 1.2 us.)  A record is two words: kRecDist holds the dist of the
// member's key (0xffffffff: no key) under a 32-bit tag, kRecRest the rest of the
// record (rec_rest) under a 21-bit tag.  The last two words are unused.
enum { kRecDist = 0, kRecRest = 1, kRecFields = 4 };
__host__ __device__ inline uint64_t* rec_word(uint64_t* recs, int nwg, uint32_t slot, int field, int g) {
    (void)nwg;
    return recs + ((size_t)g * 2 + slot) * kRecFields + (size_t)field;
}

// The second word of a record: the lowest vertex of the member's key (24 bits:
// at most 1024 members of at most 16384 columns), the number of its columns at
// that dist (15 bits), the zero-weight hazard flag, and the low 21 bits of the
// tag, which tell exchange b from b - 2, the only other one whose word the slot
// can hold (or from the cleared word, before the tag first wraps).  Bit 63 stays
// clear (see exchange_stamp).
constexpr int kRestCountShift = 24, kRestZeroShift = 39, kRestTagShift = 42;
constexpr uint32_t kRestTagMask = 0x1fffffu;
__host__ __device__ constexpr uint64_t rec_rest(uint32_t tag, uint32_t vertex, uint32_t count, uint32_t zero) {
    return ((uint64_t)(tag & kRestTagMask) << kRestTagShift) | ((uint64_t)zero << kRestZeroShift) |
           ((uint64_t)count << kRestCountShift) | (vertex & 0xffffffu);
}
__host__ __device__ constexpr uint32_t rest_tag(uint64_t w) { return (uint32_t)(w >> kRestTagShift); }
__host__ __device__ constexpr uint32_t rest_vertex(uint64_t w) { return (uint32_t)w & 0xffffffu; }
__host__ __device__ constexpr uint32_t rest_count(uint64_t w) { return (uint32_t)(w >> kRestCountShift) & 0x7fffu; }
__host__ __device__ constexpr uint32_t rest_zero(uint64_t w) { return (uint32_t)(w >> kRestZeroShift) & 1u; }

template <typename X>
__device__ __forceinline__ X ld_agent(const X* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename X>
__device__ __forceinline__ void st_agent(X* p, X v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Barrier stress (the separately built libsssp_stress.so only): before it
// arrives at an exchange (its stamp or barrier arrival; in a tagged exchange,
// its list entries and, separately, its record), a workgroup pauses for a
// pseudo-random 0 to ~25 us chosen by (workgroup, key), so that tests see many
// arrival orders, late members and entries that arrive after their record; and
// after an exchange its waves but the first pause likewise before they read the
// result (stress_wave_delay), while the first goes on.  Compiled out of the
// product library.
__device__ __forceinline__ void stress_delay(uint32_t key) {
#ifdef SSSP_STRESS_DELAYS
    uint32_t h = (blockIdx.x + 1u) * 0x9E3779B9u ^ (key * 0x85EBCA6Bu);
    h ^= h >> 15;
    h *= 0x2C1B3C6Du;
    h ^= h >> 12;
    if ((h & 3u) == 0u)
        for (uint32_t i = 0, k = (h >> 8) & 7u; i < k; ++i) __builtin_amdgcn_s_sleep(127);
#else
    (void)key;
#endif
}
__device__ __forceinline__ void stress_wave_delay(uint32_t key) {
#ifdef SSSP_STRESS_DELAYS
    if (threadIdx.x >= kWave) stress_delay(key * 16u + threadIdx.x / kWave);
#else
    (void)key;
#endif
}

__device__ __forceinline__ uint64_t umin64(uint64_t a, uint64_t b) { return b < a ? b : a; }
__host__ __device__ __forceinline__ uint64_t make_key(uint32_t d, uint32_t v) {
    return ((uint64_t)d << 32) | v;
}

// Lane index within the wave, recomputed where it is used: the empty asm keeps
// the compiler from hoisting the shuffle addresses derived from it out of the
// round loops, where they would stay live (and spill) across the row streams.
__device__ __forceinline__ int wave_lane() {
    int l = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
    asm volatile("" : "+v"(l));
    return l;
}
// x of lane (lane ^ o); o < 64
__device__ __forceinline__ uint32_t xor_lane32(uint32_t x, int lane, int o) {
    return (uint32_t)__builtin_amdgcn_ds_bpermute((lane ^ o) << 2, (int)x);
}

// Wave-wide reductions and scans, which every caller runs with all 64 lanes
// active.  Inside each row of 16 lanes they use DPP row shifts (a VALU operand
// read from the lane k below, no LDS round trip: ds_bpermute chains made the
// per-round reductions cost about 1 us each); the four row results are then
// combined from lanes 15, 31, 47 and 63 with v_readlane (scalar registers).
// row_shr:k; a lane with no source lane in its row gets `old`.
template <int K>
__device__ __forceinline__ uint32_t row_shr(uint32_t old, uint32_t x) {
    static_assert(K >= 1 && K <= 15, "row_shr:1..15");
    return (uint32_t)__builtin_amdgcn_update_dpp((int)old, (int)x, 0x110 + K, 0xf, 0xf, false);
}
template <int K>
__device__ __forceinline__ uint64_t row_shr64(uint64_t x) {  // a lane with no source keeps x
    return ((uint64_t)row_shr<K>((uint32_t)(x >> 32), (uint32_t)(x >> 32)) << 32) |
           row_shr<K>((uint32_t)x, (uint32_t)x);
}
__device__ __forceinline__ uint32_t lane_value(uint32_t x, int l) {
    return (uint32_t)__builtin_amdgcn_readlane((int)x, l);
}
__device__ __forceinline__ uint64_t lane_value64(uint64_t x, int l) {
    return ((uint64_t)lane_value((uint32_t)(x >> 32), l) << 32) | lane_value((uint32_t)x, l);
}

// A value that is the same in every lane, moved to a scalar register (so that
// branches and loops on it are scalar).
__device__ __forceinline__ uint32_t scalar(uint32_t x) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)x); }

// minimum over the wave, in every lane
__device__ __forceinline__ uint64_t wave_min64(uint64_t x) {
    x = umin64(x, row_shr64<1>(x));
    x = umin64(x, row_shr64<2>(x));
    x = umin64(x, row_shr64<4>(x));
    x = umin64(x, row_shr64<8>(x));  // lane 15 of each row: the row's minimum
    return umin64(umin64(lane_value64(x, 15), lane_value64(x, 31)), umin64(lane_value64(x, 47), lane_value64(x, 63)));
}
// OR over the wave, in every lane
__device__ __forceinline__ uint32_t wave_or32(uint32_t x) {
    x |= row_shr<1>(0u, x);
    x |= row_shr<2>(0u, x);
    x |= row_shr<4>(0u, x);
    x |= row_shr<8>(0u, x);
    return lane_value(x, 15) | lane_value(x, 31) | lane_value(x, 47) | lane_value(x, 63);
}
// inclusive prefix sum over the wave
__device__ __forceinline__ uint32_t wave_scan32(uint32_t x) {
    x += row_shr<1>(0u, x);
    x += row_shr<2>(0u, x);
    x += row_shr<4>(0u, x);
    x += row_shr<8>(0u, x);  // prefix within the row
    const uint32_t r0 = lane_value(x, 15), r1 = lane_value(x, 31), r2 = lane_value(x, 47);
    const int row = wave_lane() >> 4;
    return x + (row >= 1 ? r0 : 0u) + (row >= 2 ? r1 : 0u) + (row >= 3 ? r2 : 0u);
}

// The same for 32-bit values, in six DPP steps and one v_readlane: the rows'
// results are passed on by row_bcast15 / row_bcast31 (lane 15 of a row to the
// next row, lane 31 to the upper half), so that lane 63 ends with the wave's.
// A DPP operand needs no 64-bit compare and select: with reductions over 64-bit
// keys a round of the whole-GPU solve (n=16384) took 1.1 us to publish and 0.8 us
// to reduce the records, with these and ballots 0.5 and 0.4 to 0.6 us (one wave
// runs straight-line code at about ten cycles an instruction).
template <int CTRL, int ROWS>
__device__ __forceinline__ uint32_t dpp32(uint32_t old, uint32_t x) {
    return (uint32_t)__builtin_amdgcn_update_dpp((int)old, (int)x, CTRL, ROWS, 0xf, false);
}
__device__ __forceinline__ uint32_t wave_min32(uint32_t x) {
    x = min(x, dpp32<0x111, 0xf>(~0u, x));
    x = min(x, dpp32<0x112, 0xf>(~0u, x));
    x = min(x, dpp32<0x114, 0xf>(~0u, x));
    x = min(x, dpp32<0x118, 0xf>(~0u, x));
    x = min(x, dpp32<0x142, 0xa>(~0u, x));  // row_bcast15 into rows 1 and 3
    x = min(x, dpp32<0x143, 0xc>(~0u, x));  // row_bcast31 into rows 2 and 3
    return lane_value(x, kWave - 1);
}
__device__ __forceinline__ uint32_t wave_prefix32(uint32_t x) {  // inclusive prefix sum
    x += dpp32<0x111, 0xf>(0u, x);
    x += dpp32<0x112, 0xf>(0u, x);
    x += dpp32<0x114, 0xf>(0u, x);
    x += dpp32<0x118, 0xf>(0u, x);
    x += dpp32<0x142, 0xa>(0u, x);
    x += dpp32<0x143, 0xc>(0u, x);
    return x;
}
__device__ __forceinline__ uint64_t wave_mask(bool b) { return __builtin_amdgcn_ballot_w64(b); }
// set bits of a wave mask below this lane
__device__ __forceinline__ uint32_t lanes_below(uint64_t m) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// LDS scratch for block-wide reductions (one slot per wave).
template <int T>
struct Red {
    uint64_t k[T / kWave];
    uint32_t a[T / kWave];
    uint32_t b[T / kWave];
};

// Block-wide min of a 64-bit key and OR of 32-bit flags; every thread gets both.
template <int T>
__device__ __forceinline__ void block_min_or(uint64_t& key, uint32_t& flags, Red<T>& red) {
    key = wave_min64(key);
    flags = wave_or32(flags);
    const int w = threadIdx.x / kWave;
    if ((threadIdx.x & (kWave - 1)) == 0) {
        red.k[w] = key;
        red.a[w] = flags;
    }
    __syncthreads();
    key = red.k[0];
    flags = red.a[0];
#pragma unroll
    for (int i = 1; i < T / kWave; ++i) {
        key = umin64(key, red.k[i]);
        flags |= red.a[i];
    }
    __syncthreads();
}

// Block-wide "any": true in every thread if pred is non-zero in some thread.
// Also a workgroup barrier.
template <int T>
__device__ __forceinline__ bool block_any(int pred, Red<T>& red) {
    const bool w = __builtin_amdgcn_ballot_w64(pred != 0) != 0;
    if ((threadIdx.x & (kWave - 1)) == 0) red.a[threadIdx.x / kWave] = w ? 1u : 0u;
    __syncthreads();
    uint32_t any = 0;
#pragma unroll
    for (int i = 0; i < T / kWave; ++i) any |= red.a[i];
    __syncthreads();
    return any != 0;
}

// Block-wide exclusive prefix sum; returns this thread's offset and the total.
template <int T>
__device__ __forceinline__ uint32_t block_excl_scan(uint32_t x, uint32_t& total, Red<T>& red) {
    const uint32_t inc = wave_scan32(x);
    const int w = threadIdx.x / kWave;
    if ((threadIdx.x & (kWave - 1)) == kWave - 1) red.b[w] = inc;
    __syncthreads();
    uint32_t before = 0, tot = 0;
#pragma unroll
    for (int i = 0; i < T / kWave; ++i) {
        const uint32_t s = red.b[i];
        if (i < w) before += s;
        tot += s;
    }
    __syncthreads();
    total = tot;
    return before + inc - x;
}

// Thread -> (row partition, lane) layout for a slice of S columns.
struct Layout {
    int L;   // lanes per row (power of two, <= T)
    int P;   // row partitions (T / L)
    int r;   // this thread's partition
    int c;   // this thread's lane
    int NG;  // column groups of 4 in the slice
};

template <int T>
__device__ __forceinline__ Layout make_layout(int S) {
    Layout lo;
    lo.NG = (S + 3) >> 2;
    int L = 1;
    while (L < lo.NG && L < T) L <<= 1;
    lo.L = L;
    lo.P = T / L;
    lo.r = threadIdx.x / L;
    lo.c = threadIdx.x % L;
    return lo;
}


// Matrix entries as stored.  int32_t is the caller's matrix (INT32_MAX = no
// edge).  uint16_t / uint8_t are exact compact copies that the library builds
// of a graph it will stream many times, when every finite weight fits below
// the type's all-ones code, which stands for "no edge".  Four consecutive
// entries (one column group) are read with one 16-, 8- or 4-byte load and
// widened to uint32 with the no-edge code mapped back to INT32_MAX.
template <typename E>
__device__ __forceinline__ uint32_t widen(uint32_t v);
template <>
__device__ __forceinline__ uint32_t widen<int32_t>(uint32_t v) { return v; }
template <>
__device__ __forceinline__ uint32_t widen<uint16_t>(uint32_t v) { return v == 0xffffu ? kInf : v; }
template <>
__device__ __forceinline__ uint32_t widen<uint8_t>(uint32_t v) { return v == 0xffu ? kInf : v; }

// Per-column candidate key of a round: the lexicographic minimum over the
// streamed rows u of (weight, u).  For the caller's int32 matrix a 64-bit key
// (W[u][v] << 32) | u.  For compact copies (n <= 65536) a 32-bit key
// (code << 16) | u built from the stored code itself: the no-edge code (all
// ones) sorts above every weight, so nothing is widened while streaming (3
// vector operations per entry: extract, shift-or, 32-bit minimum, instead of
// about 8 with widened 64-bit keys) and a lane's keys take half the registers.
template <typename E>
struct KeyOf {
    typedef uint64_t type;
};
template <>
struct KeyOf<uint16_t> {
    typedef uint32_t type;
};
template <>
struct KeyOf<uint8_t> {
    typedef uint32_t type;
};
template <typename E>
using key_t = typename KeyOf<E>::type;

template <typename E>
__device__ __forceinline__ key_t<E> key_none() {
    return (key_t<E>)~(key_t<E>)0;
}
// Key of an entry as read (the int32 bits, or the compact code) in row u.
template <typename E>
__device__ __forceinline__ key_t<E> key_make(uint32_t raw, uint32_t u) {
    if constexpr (sizeof(E) == 4) return ((uint64_t)raw << 32) | u;
    else return (raw << 16) | u;
}
// Weight of a key: INT32_MAX for no edge (and for the no-key value of compact
// keys); an int32 key above INT32_MAX holds a negative weight (or is no key).
template <typename E>
__device__ __forceinline__ uint32_t key_weight(key_t<E> k) {
    if constexpr (sizeof(E) == 4) {
        return (uint32_t)(k >> 32);
    } else {
        const uint32_t code = k >> 16;
        return code >= (uint32_t)(E)~(E)0 ? kInf : code;
    }
}
template <typename E>
__device__ __forceinline__ uint32_t key_row(key_t<E> k) {
    if constexpr (sizeof(E) == 4) return (uint32_t)k;
    else return k & 0xffffu;
}
template <typename X>
__device__ __forceinline__ X key_min(X a, X b) {
    return b < a ? b : a;
}

// Columns of the slice held by one thread: G groups of 4.  dist and pred stay in
// registers for the whole solve and are written out once at the end (a8), so no
// per-column output address is kept live across the rounds.  x is a column's
// dist (at most INT32_MAX) while it is open, and with kSettled set once it is
// settled; 0xffffffff for a position that is no column of the slice or matrix,
// or that another thread owns.  So one unsigned comparison tells an open column,
// a settled one never wins a minimum, and there is no visited mask to test.
constexpr uint32_t kSettled = 0x80000000u;
template <int G, typename E = int32_t>
struct Cols {
    uint32_t x[G][4];
    int32_t pred[G][4];
    key_t<E> best[G][4];
};

// The matrix always lives in global memory (device or pinned host memory).
// Descriptors loaded from memory carry generic pointers, which the compiler
// would access with FLAT instructions; casting to the global address space
// makes the row loads plain global loads.
// (The host pass of the same source has no address spaces.)
#if defined(__HIP_DEVICE_COMPILE__)
template <typename T>
using global_ptr = const __attribute__((address_space(1))) T*;
#else
template <typename T>
using global_ptr = const T*;
#endif

// One column group as loaded (16, 8 or 4 bytes) and its widening to uint32.
// Rows of the caller's int32 matrix start at any multiple of 4 bytes (an odd n
// or row stride): the hardware takes a 16-byte load there, so the type carries
// that alignment and every stride has the same loads.  (With one load per entry
// for rows not 16-byte aligned, n=5001 took 166 us, now 125, and a batch of 24
// graphs of any n up to 6000, one workgroup each, 7.2 ms, now 2.6.)  Rows of compact
// copies are multiples of 16 entries.
template <typename E>
struct Raw;
typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v4i_any __attribute__((ext_vector_type(4), aligned(4)));
typedef unsigned v2u __attribute__((ext_vector_type(2)));
template <>
struct Raw<int32_t> {
    typedef v4i_any type;
};
template <>
struct Raw<uint16_t> {
    typedef v2u type;
};
template <>
struct Raw<uint8_t> {
    typedef uint32_t type;
};

template <typename E>
__device__ __forceinline__ void unpack(const typename Raw<E>::type& x, uint32_t (&w)[4]);
template <>
__device__ __forceinline__ void unpack<int32_t>(const v4i_any& x, uint32_t (&w)[4]) {
    w[0] = (uint32_t)x.x;
    w[1] = (uint32_t)x.y;
    w[2] = (uint32_t)x.z;
    w[3] = (uint32_t)x.w;
}
// Compact entries stay as codes (see key_make).
template <>
__device__ __forceinline__ void unpack<uint16_t>(const v2u& x, uint32_t (&w)[4]) {
    w[0] = x.x & 0xffffu;
    w[1] = x.x >> 16;
    w[2] = x.y & 0xffffu;
    w[3] = x.y >> 16;
}
template <>
__device__ __forceinline__ void unpack<uint8_t>(const uint32_t& x, uint32_t (&w)[4]) {
    w[0] = x & 0xffu;
    w[1] = (x >> 8) & 0xffu;
    w[2] = (x >> 16) & 0xffu;
    w[3] = x >> 24;
}

// A group of 4 columns of which only the first 4 - s exist (the last one of an
// int32 matrix whose n is not a multiple of 4) is read as the 4 columns that end
// with the row, s columns to the left of its own: its keys are moved up by s
// before a pass over the rows and back down after it, which drops the
// neighbour's.  Compact copies need no shift: their rows are padded with the
// no-edge code.
template <typename E>
__device__ __forceinline__ int group_shift(int v0, int width) {
    return sizeof(E) == 4 ? max(0, v0 + 4 - width) : 0;
}
template <typename X>
__device__ __forceinline__ void shift_up(X (&v)[4], int s, X none) {
    if (s & 1) {
        v[3] = v[2];
        v[2] = v[1];
        v[1] = v[0];
        v[0] = none;
    }
    if (s & 2) {
        v[3] = v[1];
        v[2] = v[0];
        v[1] = v[0] = none;
    }
}
template <typename X>
__device__ __forceinline__ void shift_down(X (&v)[4], int s, X none) {
    if (s & 1) {
        v[0] = v[1];
        v[1] = v[2];
        v[2] = v[3];
        v[3] = none;
    }
    if (s & 2) {
        v[0] = v[2];
        v[1] = v[3];
        v[2] = v[3] = none;
    }
}

// Rows list[i], list[i + step], ... (U of them) of one column group (4 columns
// starting at p0 within each row) into `best`; past the end of the list its last
// row is repeated (a duplicate cannot change a minimum).  NT: the loads carry
// the nontemporal hint, for matrices streamed once per solve (the whole-GPU
// solve) rather than reused from the caches across instances.
template <int U, typename E, bool NT, typename R>
__device__ __forceinline__ void stream_batch(key_t<E> (&best)[4], const E* __restrict__ p0, int64_t ld,
                                             const R* list, int m, int i, int step) {
    uint32_t uu[U];
#pragma unroll
    for (int q = 0; q < U; ++q) {
        const int idx = i + q * step;
        uu[q] = (uint32_t)list[idx < m ? idx : m - 1];
    }
    // issue all U loads before using any of them: keeps U rows in flight per thread
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
        uint32_t w[4];
        unpack<E>(raw[q], w);
#pragma unroll
        for (int j = 0; j < 4; ++j) best[j] = key_min(best[j], key_make<E>(w[j], uu[q]));
    }
}

// Rows list[first], list[first + step], ... of one column group, U in flight,
// for the partitions first = 0 .. step - 1.  A list that gives a partition only
// one or two rows (small rounds) is read in a batch of that size: with eight loads
// of the same row a one-row round's stream took 1.2 us, with one 0.8 us (n=4096,
// 64 workgroups).
template <int U, typename E, bool NT, typename R>
__device__ __forceinline__ void stream_group(key_t<E> (&best)[4], const E* __restrict__ p0, int64_t ld,
                                             const R* list, int m, int first, int step) {
    if (m <= 2 * step) {
        if (first >= m) return;
        if (m <= step) stream_batch<1, E, NT>(best, p0, ld, list, m, first, step);
        else stream_batch<2, E, NT>(best, p0, ld, list, m, first, step);
        return;
    }
    for (int i = first; i < m; i += step * U) stream_batch<U, E, NT>(best, p0, ld, list, m, i, step);
}

// Can a row of a round of dist d lower one of a group's 4 columns?  Only an open
// column above d + wmin, the smallest weight known (0 for the caller's matrices:
// weights are not negative and an improvement is strict).  (One subtraction per column: values up to d + wmin wrap to the top,
// settled ones and those that are no column come out above the open ones.)
__device__ __forceinline__ bool group_open(const uint32_t (&x)[4], uint32_t d, uint32_t wmin) {
    const uint32_t lim = d + wmin;
    const uint32_t t = min(min(x[0] - (lim + 1u), x[1] - (lim + 1u)), min(x[2] - (lim + 1u), x[3] - (lim + 1u)));
    return lim < kInf && t < kInf - lim;
}
template <int G>
__device__ __forceinline__ uint32_t groups_open(const uint32_t (&x)[G][4], uint32_t d, uint32_t wmin) {
    uint32_t m = 0;
#pragma unroll
    for (int k = 0; k < G; ++k) m |= (group_open(x[k], d, wmin) ? 1u : 0u) << k;
    return m;
}

// Stream rows list[r], list[r + P], ... (m entries in `list`, partition r) of
// the matrix restricted to the slice into the running per-column minima, U rows
// in flight per thread.  `width` = columns of the slice that exist in the
// matrix (<= S).
template <int G, int U, typename E, bool NT = false, typename R = int32_t>
__device__ __forceinline__ void stream_rows(Cols<G, E>& cs, const Layout& lo, const E* __restrict__ W,
                                            int64_t ld, int64_t col0, int width, const R* list, int m) {
    // One column group at a time keeps only U x 4 weights live per thread.
#pragma unroll
    for (int k = 0; k < G; ++k) {
        const int v0 = 4 * (lo.c + k * lo.L);
        if (v0 >= width) continue;
        const int s = group_shift<E>(v0, width);
        if (col0 + v0 < s) {  // a matrix of fewer than 4 columns
            for (int i = lo.r; i < m; i += lo.P)
                for (int j = 0; j < 3; ++j)
                    if (j < width)
                        cs.best[k][j] = key_min(cs.best[k][j], key_make<E>((uint32_t)W[(int64_t)list[i] * ld + j],
                                                                           (uint32_t)list[i]));
            continue;
        }
        if (s) shift_up(cs.best[k], s, key_none<E>());
        stream_group<U, E, NT>(cs.best[k], W + (col0 + v0 - s), ld, list, m, lo.r, lo.P);
        if (s) shift_down(cs.best[k], s, key_none<E>());
    }
}

// Rounds of many rows with few groups left to lower (the stragglers of a dense
// graph): the workgroup's threads take a row each instead of a group each, so
// that 64 lanes of a wave are at work on one group and not one.  By rows, a
// partition waits for its rows in batches of 8, about m / 12 P microseconds
// (measured: 0.7 us a batch); by groups, about 1 + m / 2048 for each of the ng.
// (n=65536, p=0.5, sources with a few vertices beyond the large last bucket:
// 2.5 ms without, 1.2 with.)
// `bytes`: of the slice's part of a row, where all workgroups of the GPU read at once and
// the memory's rate bounds them (else all ones): a group's 16 bytes cost a line of 128,
// and rows are read by groups only while these come to less than the part whole (n=33000,
// p=0.05, ten of 33 groups left: 602 us whole, 938 by groups).  A gang among others is
// bound by its waits (a plan of 62 compact instances, slices of 928 columns: 180 us,
// under this limit too 241).
constexpr uint32_t kSparseGroups = 16;
constexpr uint32_t kLineBytes = 128;
__host__ __device__ __forceinline__ bool sparse_round(uint32_t ng, uint32_t m, int P, uint32_t bytes) {
    return ng <= kSparseGroups && m > 64u && ng * kLineBytes <= bytes &&
           (uint64_t)ng * (2048u + m) * (12u * (uint32_t)P) < (uint64_t)m * 2048u;
}

// One group (its 4 columns starting at local column v0) of such a round: row(e)
// is the e-th of the m rows; the group's four keys go to out[0..3] (LDS, all
// ones between rounds).
template <int T, typename E, bool NT, typename Row>
__device__ __forceinline__ void stream_sparse(const E* __restrict__ W, int64_t ld, int64_t col0, int width, int v0,
                                              int m, Row row, key_t<E>* out) {
    constexpr int U = 4;
    const int s = group_shift<E>(v0, width);
    const E* p0 = W + (col0 + v0 - s);  // m > 64 rows: at least 4 columns
    key_t<E> best[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) best[j] = key_none<E>();
    for (int i = (int)threadIdx.x; i < m; i += T * U) {
        uint32_t uu[U];
#pragma unroll
        for (int q = 0; q < U; ++q) uu[q] = row(min(i + q * T, m - 1));
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
            uint32_t w[4];
            unpack<E>(raw[q], w);
#pragma unroll
            for (int j = 0; j < 4; ++j) best[j] = key_min(best[j], key_make<E>(w[j], uu[q]));
        }
    }
    if (s) shift_down(best, s, key_none<E>());
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        key_t<E> b;
        if constexpr (sizeof(E) == 4) b = wave_min64(best[j]);
        else b = wave_min32(best[j]);
        if (wave_lane() == 0)
            __hip_atomic_fetch_min(&out[j], b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
}

// Merge the P partitions' minima into the owner threads (partition 0): every
// partition takes an LDS atomic minimum into one key per column, then the
// owners read the result and put the all-ones key back.  `mrg` (4 * L keys or
// more) is all ones between merges (clear_merge at the start of a solve).
// Only used when P > 1, which implies G == 1.
template <int T, int G, typename E>
__device__ __forceinline__ void merge_partitions(Cols<G, E>& cs, const Layout& lo, uint64_t* mrg) {
    if (lo.P == 1) return;
    key_t<E>* m = reinterpret_cast<key_t<E>*>(mrg);  // all-ones keys of either width
#pragma unroll
    for (int j = 0; j < 4; ++j)
        if (cs.best[0][j] != key_none<E>())
            __hip_atomic_fetch_min(&m[j * lo.L + lo.c], cs.best[0][j], __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_WORKGROUP);
    __syncthreads();
    if (lo.r == 0) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            cs.best[0][j] = m[j * lo.L + lo.c];
            m[j * lo.L + lo.c] = key_none<E>();
        }
    }
}

// Fill the partition-merge area (n64 keys) with all ones; ordered before its
// first use by the workgroup barriers that precede any merge.
template <int T>
__device__ __forceinline__ void clear_merge(uint64_t* mrg, int n64) {
    for (int i = threadIdx.x; i < n64; i += T) mrg[i] = kNoKey;
}

// Exclusive prefix sum over the slice owners (the first L threads, partition 0); valid
// in the owners, `total` gets the sum.  Threads that are not owners must pass 0.  When
// the owners fit in wave 0 this is a wave scan with no workgroup barrier (and only wave
// 0 takes part); otherwise a block scan that every thread must enter.
template <int T>
__device__ __forceinline__ uint32_t owner_excl_scan(uint32_t x, uint32_t& total, int L, Red<T>& red) {
    if (L <= kWave) {
        uint32_t inc = 0;
        if (threadIdx.x < kWave) {
            inc = wave_scan32(x);
            total = (uint32_t)__builtin_amdgcn_readlane((int)inc, kWave - 1);
        }
        return inc - x;
    }
    return block_excl_scan<T>(x, total, red);
}

template <int G, typename E>
__device__ __forceinline__ void reset_best(Cols<G, E>& cs) {
#pragma unroll
    for (int k = 0; k < G; ++k)
#pragma unroll
        for (int j = 0; j < 4; ++j) cs.best[k][j] = key_none<E>();
}

// Local vertex index of (k, j) for this thread.
__device__ __forceinline__ int local_col(const Layout& lo, int k, int j) {
    return 4 * (lo.c + k * lo.L) + j;
}

// Initialise the owned columns: dist = inf (0 at the source), pred = -1, open.
template <int G, typename E>
__device__ __forceinline__ void init_cols(Cols<G, E>& cs, const Layout& lo, int64_t col0, int width,
                                          int32_t src) {
#pragma unroll
    for (int k = 0; k < G; ++k)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int v = local_col(lo, k, j);
            const bool mine = lo.r == 0 && k * lo.L + lo.c < lo.NG && v < width;
            cs.x[k][j] = !mine ? 0xffffffffu : col0 + v == src ? 0u : kInf;
            cs.pred[k][j] = -1;
        }
    reset_best(cs);
}

// Settle the open columns at dist d (the round's bucket), or, with `step`, only
// the one whose bit is in `only`; the mask of the columns settled.
template <int G, typename E>
__device__ __forceinline__ uint32_t settle(Cols<G, E>& cs, uint32_t d, bool step, uint32_t only) {
    uint32_t m = 0;
#pragma unroll
    for (int k = 0; k < G; ++k)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint32_t bit = 1u << (4 * k + j);
            const bool take = cs.x[k][j] == d && (!step || (only & bit));
            if (take) m |= bit;
            cs.x[k][j] |= take ? kSettled : 0u;
        }
    return m;
}

// Undo settle for the columns of its mask (a discarded round).
template <int G, typename E>
__device__ __forceinline__ void reopen(Cols<G, E>& cs, uint32_t mask) {
#pragma unroll
    for (int k = 0; k < G; ++k)
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (mask >> (4 * k + j) & 1u) cs.x[k][j] &= ~kSettled;
}

// Candidate dist of a column from the round's minimum key (d + min weight);
// returns kInf + something >= dist when there is no usable edge.  Sets *neg if
// the minimum weight read as uint32 exceeds INT32_MAX (a negative weight).
template <typename E>
__device__ __forceinline__ uint32_t candidate(key_t<E> best, uint32_t d, uint32_t& neg) {
    const uint32_t w = key_weight<E>(best);
    if (w > kInf) {
        neg |= best != key_none<E>() ? kStatusNegWeight : 0u;
        return 0xffffffffu;
    }
    return d + w;  // d < 2^31-1 and w <= 2^31-1: no wrap
}

// Dist of the open columns if the pending round (bucket dist d) is applied; a
// position that is not open keeps its x, which is above every dist.  `neg` gets
// its sign bit set if a negative weight was the best candidate of a column, in a
// round that read rows (`met`): every open column above d has then met one, so its
// key is a weight's.
// With the bucket settled beforehand, a candidate equal to d exists exactly when
// the bucket has a zero-weight edge to an open vertex outside it: such a vertex
// would join the bucket during the round and change the order Algorithm 1
// settles it in (the zero-weight hazard of a fused round).
template <int G, typename E>
__device__ __forceinline__ void candidates(const Cols<G, E>& cs, uint32_t d, bool met, uint32_t (&cand)[G][4],
                                           uint32_t& neg) {
#pragma unroll
    for (int k = 0; k < G; ++k)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint32_t x = cs.x[k][j], w = key_weight<E>(cs.best[k][j]);
            // saturating: a weight above INT32_MAX (a negative one) offers nothing
            cand[k][j] = (int32_t)x >= 0 ? min(x, __builtin_elementwise_add_sat(d, w)) : x;
            neg |= met ? w & ~x : 0u;
        }
}

// Apply a round: every open column takes its candidate if strictly smaller
// (pred = the candidate's row).
template <int G, typename E>
__device__ __forceinline__ void commit(Cols<G, E>& cs, const uint32_t (&cand)[G][4]) {
#pragma unroll
    for (int k = 0; k < G; ++k)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (cand[k][j] < cs.x[k][j]) cs.pred[k][j] = (int32_t)key_row<E>(cs.best[k][j]);
            cs.x[k][j] = cand[k][j];
        }
    reset_best(cs);
}

// Write the owned dist and pred values out (a8: writeback): one 16-byte store
// per column group and array where the group is whole and aligned.
template <int G, typename E>
__device__ __forceinline__ void write_out(const Cols<G, E>& cs, const Layout& lo, int64_t col0, int width,
                                          int32_t* __restrict__ dist, int32_t* __restrict__ pred) {
    if (lo.r != 0) return;
#pragma unroll
    for (int k = 0; k < G; ++k) {
        if (k * lo.L + lo.c >= lo.NG) continue;
        const int v0 = local_col(lo, k, 0);
        int32_t* dp = dist + col0 + v0;
        int32_t* pp = pred + col0 + v0;
        if (v0 + 3 < width && (((uintptr_t)dp | (uintptr_t)pp) & 15u) == 0) {
            *reinterpret_cast<v4i*>(dp) = v4i{(int)(cs.x[k][0] & kInf), (int)(cs.x[k][1] & kInf),
                                              (int)(cs.x[k][2] & kInf), (int)(cs.x[k][3] & kInf)};
            *reinterpret_cast<v4i*>(pp) = v4i{cs.pred[k][0], cs.pred[k][1], cs.pred[k][2], cs.pred[k][3]};
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (v0 + j < width) {
                    dp[j] = (int32_t)(cs.x[k][j] & kInf);
                    pp[j] = cs.pred[k][j];
                }
        }
    }
}

}  // namespace sssp
