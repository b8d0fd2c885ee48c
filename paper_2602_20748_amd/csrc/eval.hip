// Plain RPQ evaluation: multi-source, level-synchronous search of the product
// of the graph and an epsilon-free NFA, to the fixpoint.
//
// Semantics (Definition 1 with the automata-based evaluation of Section 2.2):
// from each source s the search reaches product vertices (v, q); reaching a
// final q at v puts (s, v) in the result.  A visited set of (vertex, state)
// pairs per source keeps every product vertex expanded once per source.
//
// Bit-parallel layout.  Sources are taken W = 64*K at a time (a "unit", the
// counterpart of the paper's start-vertex batch, Section 4.1).  Sources without an edge that an
// initial state can follow reach nothing: they get no bit, only their zero-length walk is counted.
// For a unit, every product vertex (q, v) that some label can lead to owns a row of K 64-bit
// words (see "rows" below); bit i of word k stands for source 64*k + i.  Per unit:
//   Vis [R][K]  bits already reached (the per-source visited sets)
//   Next[R][K]  bits reached in the level being expanded (or Vis as of the last level)
//   Touch[R]    1 while a row already sits on the next frontier list
// The answer bits of a vertex are the OR of its rows of final states.
// G units advance together; their rows are tagged by a slot id.
//
// One level = three kernels:
//   expand    every frontier entry (q, v) owns a flattened item space: its edges over the
//             labels q can follow, each counted once per successor state.  For each item
//             (edge v -l-> w, successor q') it ORs the entry's frontier bits that are new for
//             (q', w) into Next; the first writer of a row sets its touch bit.  Entries with
//             at most H items are expanded straight from the frontier list; larger ones
//             arrive as slices of at most H items (edge-balanced work whatever the degree
//             skew, with slice memory bounded by 2 * items / H).  Items whose target row is full
//             -- it holds every source that still had a bit in the last frontier but one -- are
//             dropped before the row is read.
//   compact   the touched rows become the next frontier list (ballot/popcount prefix).
//   finalize  for each new entry moves Next into a compact frontier row, ORs it into Vis,
//             counts the product edges it will examine, and cuts entries of more than H items
//             into slices.
// The fixpoint is reached when a level appends nothing; the host checks the
// list counter every few levels (no hop bound).
//
// Extraction walks the answer bits: per source its count and checksum, and optionally the
// result keys (s << 32) | v written source-major with ascending v, so the
// output is sorted and distinct by construction.
#include "internal.h"

#include <algorithm>
#include <cstring>
#include <mutex>
#include <type_traits>
#include <utility>
#include <vector>

namespace {

constexpr int kBlock = 256;
constexpr int kWaves = kBlock / 64;

// counters[] slots (uint64)
constexpr int C_LIST = 0;       // [0..1] list length per parity
constexpr int C_DESC = 2;       // [2..3] slice count per parity
constexpr int C_ERR = 6;        // capacity / validation error flags
constexpr int C_PAIRBASE = 7;   // global key index where the current group starts
constexpr int C_COUNT = 8;
constexpr int C_HASH = 9;
constexpr int C_LASTLEVEL = 10; // 1 + highest level index whose finalize appended rows (this group)
constexpr int C_ALIVE = 11;     // sources that got a bit
constexpr int C_TALLY = 12;     // [kTallies] the work tallies below, summed over the level kernels' blocks

// Work tallies of the level kernels.  Every block keeps its own copy (blocks of one launch write
// disjoint lines, launches follow each other on the stream), and k_tally_sum adds the copies up once
// per call.  One atomic per wave to shared counters cost more than it looked: the 20,000 or more
// same-line atomics of a launch complete one after another: when they were taken out, a 2,500-source
// slice of R-MAT 18 with keys went from 6.10 to 3.97 ms (it takes 1.7 since) and every launch of k_expand
// on R-MAT 18 lost 0.06 ms.
constexpr int T_ITEMS = 0;      // expansion (profiling)
constexpr int T_DESCS = 1;
constexpr int T_WREAD = 2;
constexpr int T_WUPD = 3;
constexpr int T_EPROD = 4;      // finalize: product edges examined,
constexpr int T_FROWS = 5;      //   (profiling) rows finalized,
constexpr int T_FWORDS = 6;     //   and their non-zero Next words
constexpr int T_FFRESH = 7;     //   rows listed for the first time
constexpr int kTallies = 8;
constexpr int kTallyStride = 8;             // words per block
constexpr unsigned kMaxLevelBlocks = 2048;  // upper bound of a level kernel's grid
constexpr unsigned kMaxExtractBlocks = 4096;  // and of an extraction that keeps totals per block
constexpr int C_NCOUNTERS = C_TALLY + kTallies;

constexpr uint64_t ERR_LIST = 1, ERR_DESC = 2, ERR_SOURCES = 4;

// A slice [beg, beg + len) of the item space of frontier entry `entry` (an entry with more than
// H items is cut into such slices of at most H items).
struct Desc {
    uint32_t entry, len;
    uint64_t beg;
};

// Rows.  A slot has R rows; those of state q are [base[q], base[q + 1]):
//   ROW_ALL     row base + v for every vertex v
//   ROW_RANKED  one row for each vertex of a class, the vertices that q's entering labels can lead to
//               (and the sources, for an initial state): row base + (rank of v in the class)
//   ROW_SOURCE  q is initial and nothing leads back to it: row base + j for source j of the unit
// Bitmaps are cleared, and final rows extracted, for every group of units, so rows that no walk can reach
// cost as much as the others: of R-MAT 23's 8.4M vertices a given label leads to a fifth, and an initial
// state of 4,096 sources needs 4,096 rows.  A rank costs one 16-byte read of a table that stays in L2
// (2 MB a class there), so classes are used where the bitmaps are large (kCompactBytes) and the class
// leaves out at least a quarter of the vertices.
enum RowKind : uint32_t { ROW_ALL = 0, ROW_RANKED = 1, ROW_SOURCE = 2 };

constexpr uint32_t kNone = 0xFFFFFFFFu;

struct DevNfa {
    uint32_t Q, L, init, final;
    uint32_t base[RPQ_MAX_STATES + 1];
    uint32_t kind[RPQ_MAX_STATES];
    uint32_t rank_at[RPQ_MAX_STATES];   // ROW_RANKED: its class's first word in Args::rank
    uint64_t list_at[RPQ_MAX_STATES];   //             its class's first vertex in Args::verts
    uint64_t qlab[RPQ_MAX_STATES];                   // labels with a transition out of q
    // answers: the vertices to look at (every vertex, or a class) and where sources rank (kNone: no
    // ROW_SOURCE state is final)
    uint32_t ans_class, ans_rank_at, src_rank_at;
    uint64_t ans_list_at;
    uint32_t delta[RPQ_MAX_STATES * RPQ_MAX_LABELS]; // compact [q * L + l]
};

struct Args {
    const uint32_t* row_ptr;
    const uint32_t* dst;
    const uint64_t* lmask;
    const DevNfa* nfa;
    const ulonglong2* rank;   // per class and 64 vertices: {member bits, members before them}
    const uint32_t* verts;    // per class: its vertices, ascending
    const uint32_t* class_n;  // per class: how many
    const uint32_t* srcs;     // sources that have a bit, in bit order, or null: 0, 1, ...
    const uint32_t* pos;      // their positions in the caller's list, or null: the same
    const uint32_t* bit_of;   // bit, within its group, of each in ascending order, or null: the same order
    uint64_t n_srcs, gbase;   // how many; the first one of the group
    uint64_t* vis;          // visited bits (with seen_or: also those found at the current level)
    uint64_t* next;         // two reads: bits found at this level; seen_or: Vis as of the last finalize
    uint64_t* touch;        // one bit per row: row has bits new at this level
    uint64_t* ever;         // seen_or: at this level or before, in the group
    uint64_t* fresh;        // seen_or: of the rows listed now, those listed for the first time
    uint8_t* full;          // per row: no source still searching can add to it
    uint64_t* active;       // [2][G][K] by list parity: sources with a bit in that frontier, or more
    uint64_t* rows0;
    uint64_t* rows1;
    uint32_t* ids0;         // row ids of the frontier lists (row = slot * R + row within the slot)
    uint32_t* ids1;
    Desc* desc0;
    Desc* desc1;
    unsigned long long* counters;
    unsigned long long* tally;    // [kMaxLevelBlocks][kTallyStride]
    unsigned long long* xtally;   // [kMaxExtractBlocks][2]: count and checksum
    const uint64_t* target;   // optional [V / 64] bitmap: only result vertices with their bit set count
    uint64_t n_active;        // G * K
    uint32_t V, L, Q, H, R, W;
    uint32_t seen_or;         // visit scheme: 0 = two reads, 1 = seen OR (see the expansion)
    uint64_t list_cap, desc_cap;
};

__device__ __forceinline__ uint64_t* rows_of(const Args& a, int p) { return p ? a.rows1 : a.rows0; }
__device__ __forceinline__ uint32_t* ids_of(const Args& a, int p) { return p ? a.ids1 : a.ids0; }
__device__ __forceinline__ Desc* desc_of(const Args& a, int p) { return p ? a.desc1 : a.desc0; }

// relaxed device-scope OR whose result is unused (no-return atomic)
__device__ __forceinline__ void or_relaxed(uint64_t* p, uint64_t v) {
    (void)__hip_atomic_fetch_or(reinterpret_cast<unsigned long long*>(p), (unsigned long long)v, __ATOMIC_RELAXED,
                                __HIP_MEMORY_SCOPE_AGENT);
}

// the automaton and the row map in LDS
struct LdsNfa {
    uint32_t delta[RPQ_MAX_STATES * RPQ_MAX_LABELS];
    uint64_t qlab[RPQ_MAX_STATES];
    uint64_t list_at[RPQ_MAX_STATES];
    uint32_t base[RPQ_MAX_STATES];
    uint32_t kind[RPQ_MAX_STATES];
    uint32_t rank_at[RPQ_MAX_STATES];
};

__device__ __forceinline__ void load_nfa(const Args& a, LdsNfa& s) {
    const uint32_t QL = a.Q * a.L;
    for (uint32_t i = threadIdx.x; i < QL; i += kBlock) s.delta[i] = a.nfa->delta[i];
    if (threadIdx.x < a.Q) {
        const uint32_t q = threadIdx.x;
        s.qlab[q] = a.nfa->qlab[q];
        s.list_at[q] = a.nfa->list_at[q];
        s.base[q] = a.nfa->base[q];
        s.kind[q] = a.nfa->kind[q];
        s.rank_at[q] = a.nfa->rank_at[q];
    }
    __syncthreads();
}

__device__ __forceinline__ uint32_t rank_in(const ulonglong2* rank, uint32_t rank_at, uint32_t v) {
    const ulonglong2 e = rank[rank_at + (v >> 6)];
    return (uint32_t)e.y + (uint32_t)__popcll(e.x & ((1ull << (v & 63)) - 1));
}

// row, within its slot, of state q2 (not ROW_SOURCE) at vertex w
__device__ __forceinline__ uint32_t target_row(const Args& a, const LdsNfa& s, uint32_t q2, uint32_t w) {
    return s.base[q2] + (s.kind[q2] == ROW_ALL ? w : rank_in(a.rank, s.rank_at[q2], w));
}

// slot, state and vertex of a row
__device__ __forceinline__ void row_entry(const Args& a, const LdsNfa& s, uint32_t row, uint32_t* slot, uint32_t* q_out,
                                          uint32_t* v) {
    const uint32_t sl = row / a.R, r = row - sl * a.R;
    uint32_t q = 0;   // the last state whose rows begin at or before r (a state without rows is passed over)
#pragma unroll
    for (uint32_t step = RPQ_MAX_STATES / 2; step >= 1; step >>= 1)
        if (q + step < a.Q && s.base[q + step] <= r) q += step;
    const uint32_t off = r - s.base[q];
    *slot = sl;
    *q_out = q;
    if (s.kind[q] == ROW_ALL) *v = off;
    else if (s.kind[q] == ROW_RANKED) *v = a.verts[s.list_at[q] + off];
    else {
        const uint64_t gi = a.gbase + (uint64_t)sl * a.W + off;
        *v = a.srcs ? a.srcs[gi] : (uint32_t)gi;
    }
}

// ------------------------------------------------------------------------------------------------
// level expansion.  Work comes as segments (entry, first item, item count): first every light
// entry of the frontier list whole, then the slices of the heavy ones.  Per batch of
// segments (one per lane) the work is mapped twice per 64 items:
//   item phase  lane i takes item i: finds its segment (prefix of the wave's segment lengths),
//               decodes the edge target w and successor q', and forms the target row id;
//   word phase  the wave splits into 64/K groups of K lanes; group g takes items g, g + 64/K, ...
//               and lane k of the group handles word k of the rows, so the frontier row, the
//               visited row and the Next row of an item are each read or updated as one
//               contiguous K-word access instead of K scattered ones.
// kUnroll items per group are loaded before any of them is updated (memory-level parallelism).
//
// New bits of a target word (Section 4, the visited check before the atomic update) are found in
// one of two ways, both giving the same frontier:
//   two reads  the visited word and the Next word are read; bits in neither are ORed into Next,
//              and finalize ORs each level's Next into the visited bitmap and clears Next;
//   seen OR    only the visited word is read; bits not in it are ORed into it alone.  The visited
//              bitmap then also holds the bits found so far at this level, so it filters as well as
//              the two reads together.  The second bitmap holds the visited bits as of the last
//              finalize, and finalize takes a listed row's new bits as Vis & ~that, then advances
//              it.  One read and one OR per new word, the method's own accesses; finalize reads one
//              more word per row word after a row's first time, when it writes the row whole.
//              Faster at both scales measured (five queries a step): R-MAT 23, 65,536 sources, 904
//              -> 628 ms (expansion 5.45 -> 3.36 ms a launch); R-MAT 18, all pairs, 183 -> 152 ms
//              (0.86 -> 0.67).
// ------------------------------------------------------------------------------------------------
constexpr int kUnroll = 8;

// An empty asm that takes each value as an operand.  Without it the compiler moves the arithmetic
// that consumes a conditionally loaded value into the load's own conditional block, where it must
// wait for that load: the kUnroll loads would then complete one at a time instead of together.
template <int N>
__device__ __forceinline__ void keep_in_flight(uint64_t (&x)[N]) {
#pragma unroll
    for (int u = 0; u < N; ++u) asm volatile("" : "+v"(x[u]));
}

template <int K, bool SEEN>
__device__ __forceinline__ void expand_segments(const Args& a, const LdsNfa& s, const uint64_t* rows, bool filter,
                                                bool have, uint32_t ent, uint32_t slot, uint32_t q, uint32_t v,
                                                uint64_t m, uint64_t beg, uint32_t len, uint64_t& t_items,
                                                uint64_t& t_wread, uint64_t& t_wupd) {
    constexpr int GS = 64 / K;
    const int lane = threadIdx.x & 63;
    const int grp = lane / K, k = lane % K;
    const uint64_t gmask = (K == 64) ? ~0ull : (((1ull << K) - 1) << (grp * K));
    if (!have) len = 0;
    const uint32_t incl = rpqd::wave_incl_scan_u32(len);
    const uint32_t excl = incl - len;
    const uint32_t total = __shfl(incl, 63, 64);
    if (lane == 0) t_items += total;
    for (uint32_t base = 0; base < total; base += 64) {
        // item phase
        const uint32_t item = base + lane;
        int c = 0;
#pragma unroll
        for (int step = 32; step >= 1; step >>= 1) {
            const int cand = c + step;
            const uint32_t e = __shfl(excl, cand, 64);
            if (e <= item) c = cand;
        }
        const uint32_t c_ent = __shfl(ent, c, 64);
        const uint32_t c_slot = __shfl(slot, c, 64);
        const uint32_t c_q = __shfl(q, c, 64);
        const uint32_t c_v = __shfl(v, c, 64);
        const uint64_t c_m = __shfl(m, c, 64);
        const uint64_t c_beg = __shfl(beg, c, 64);
        const uint32_t c_ex = __shfl(excl, c, 64);
        uint32_t my_row = 0;
        bool live = false;
        if (item < total) {
            uint32_t w = 0, q2 = 0;
            rpqd::decode_item(a.row_ptr, a.dst, a.L, s.delta, c_v, c_q, c_m, c_beg + (item - c_ex), &w, &q2);
            my_row = c_slot * a.R + target_row(a, s, q2, w);
            live = !SEEN || !filter || !a.full[my_row];
        }
        // live items to the front, so that the word phase sees no others
        const uint64_t lm = __ballot(live);
        const uint32_t n_here = (uint32_t)__popcll(lm);
        uint32_t my_ent = c_ent;
        if (n_here != min(64u, total - base)) {
            const uint32_t before = (uint32_t)__popcll(lm & rpqd::lanemask_lt());
            const int to = (int)(live ? before : n_here + lane - before) * 4;
            my_row = (uint32_t)__builtin_amdgcn_ds_permute(to, (int)my_row);
            my_ent = (uint32_t)__builtin_amdgcn_ds_permute(to, (int)c_ent);
        }
        // word phase
        auto words = [&](auto rows_each, uint32_t j) {
            constexpr int U = decltype(rows_each)::value;
            uint32_t r[U];
            uint64_t f[U], nb[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const uint32_t idx = j + u * GS + grp;
                r[u] = __shfl(my_row, idx & 63, 64);
                const uint32_t e = __shfl(my_ent, idx & 63, 64);
                f[u] = idx < n_here ? rows[(uint64_t)e * K + k] : 0;
            }
            if constexpr (SEEN) {
                // the visited word holds every bit of earlier levels (their ORs completed before
                // this launch): bits not in it as read are new at this level
                uint64_t sw[U];
#pragma unroll
                for (int u = 0; u < U; ++u) sw[u] = f[u] ? a.vis[(uint64_t)r[u] * K + k] : ~0ull;
                keep_in_flight<U>(sw);
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    nb[u] = f[u] & ~sw[u];
                    if (nb[u]) {
                        or_relaxed(&a.vis[(uint64_t)r[u] * K + k], nb[u]);
                    }
                }
            } else {
                // the visited word and the Next word together: bits already in Next need no OR, and
                // the OR then finds its line in L2 (Next only gains bits during an expansion, so a
                // stale copy can only let through an OR that is not needed)
                uint64_t vw[U], nx[U];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    vw[u] = f[u] ? a.vis[(uint64_t)r[u] * K + k] : ~0ull;
                    nx[u] = f[u] ? a.next[(uint64_t)r[u] * K + k] : ~0ull;
                }
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    nb[u] = f[u] & ~vw[u] & ~nx[u];
                    if (nb[u]) or_relaxed(&a.next[(uint64_t)r[u] * K + k], nb[u]);
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                t_wread += f[u] != 0;
                t_wupd += nb[u] != 0;
                const uint64_t hit = __ballot(nb[u] != 0) & gmask;
                if (k == 0 && hit) or_relaxed(&a.touch[r[u] >> 6], 1ull << (r[u] & 63));
            }
        };
        // (a step of kUnroll rows costs its instructions whether the group has them or not)
        if (SEEN && n_here <= (uint32_t)GS) words(std::integral_constant<int, SEEN ? 1 : kUnroll>(), 0);
        else
            for (uint32_t j = 0; j < n_here; j += GS * kUnroll) words(std::integral_constant<int, kUnroll>(), j);
    }
}

// Add each wave's N tallies to the block's copy, words [first, first + N).  Every thread of the block
// calls it once, at the end of the kernel.  The adds do not return: a short level waits for one access to
// memory here, not for two.
template <int N>
__device__ __forceinline__ void add_tallies(const Args& a, int first, const uint64_t (&t)[N]) {
    __shared__ uint64_t s_part[kWaves][N];
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const uint64_t x = rpqd::wave_sum_u64(t[i]);
        if ((threadIdx.x & 63) == 0) s_part[threadIdx.x >> 6][i] = x;
    }
    __syncthreads();
    if (threadIdx.x < N) {
        uint64_t x = 0;
        for (int w = 0; w < kWaves; ++w) x += s_part[w][threadIdx.x];
        if (x) atomicAdd(&a.tally[(uint64_t)blockIdx.x * kTallyStride + first + threadIdx.x], (unsigned long long)x);
    }
}

__global__ __launch_bounds__(1024) void k_tally_sum(const unsigned long long* __restrict__ tally,
                                                    const unsigned long long* __restrict__ xtally,
                                                    unsigned long long* __restrict__ counters) {
    constexpr int N = kTallies + 2;
    __shared__ uint64_t s_part[16][N];
    uint64_t t[N] = {};
    // unrolled: one block's loads all in flight together
#pragma unroll
    for (unsigned b = threadIdx.x; b < kMaxLevelBlocks; b += 1024)
#pragma unroll
        for (int i = 0; i < kTallies; ++i) t[i] += tally[(uint64_t)b * kTallyStride + i];
#pragma unroll
    for (unsigned b = threadIdx.x; b < kMaxExtractBlocks; b += 1024)
#pragma unroll
        for (int i = 0; i < 2; ++i) t[kTallies + i] += xtally[2 * (uint64_t)b + i];
    for (int i = 0; i < N; ++i) {
        const uint64_t x = rpqd::wave_sum_u64(t[i]);
        if ((threadIdx.x & 63) == 0) s_part[threadIdx.x >> 6][i] = x;
    }
    __syncthreads();
    if (threadIdx.x < N) {
        uint64_t x = 0;
        for (int w = 0; w < 16; ++w) x += s_part[w][threadIdx.x];
        if (threadIdx.x < kTallies) counters[C_TALLY + threadIdx.x] = x;
        else counters[threadIdx.x == kTallies ? C_COUNT : C_HASH] += x;
    }
}

// Entries a wave takes at a time: 64, fewer while that leaves waves without any.  A wave walks its entries'
// items 64 at a time, each step a chain of dependent reads; one source of R-MAT 18 has levels of 80,000
// entries, which at 64 are a quarter of the resident waves and 16 steps each.
__device__ __forceinline__ uint32_t batch_of(uint64_t n, uint64_t n_waves) {
    uint32_t b = 64;
    while (b > 4 && n <= n_waves * (b / 2)) b /= 2;
    return b;
}

// A list of at most this many entries a wave is short: its levels are chains of dependent accesses, with few
// full rows to gain from and one access more to see which are.  They are neither marked nor looked at there.
constexpr uint32_t kShortBatch = 4;

template <int K, bool SEEN>
__global__ __launch_bounds__(kBlock) void k_expand(Args a, int p) {
    __shared__ LdsNfa s_nfa;
    const uint64_t n_list = min((uint64_t)a.counters[C_LIST + p], a.list_cap);
    const uint64_t n_desc = min((uint64_t)a.counters[C_DESC + p], a.desc_cap);
    const uint64_t n_waves = (uint64_t)gridDim.x * kWaves, wave0 = (uint64_t)blockIdx.x * kWaves;
    const uint32_t lb = batch_of(n_list, n_waves), db = batch_of(n_desc, n_waves);
    // a short list leaves most blocks nothing to do (R-MAT 20, 1,003 sources, at most three steps: 1.44 -> 1.38 ms)
    if (n_list == 0 || (wave0 * lb >= n_list && wave0 * db >= n_desc)) return;
    load_nfa(a, s_nfa);
    const int lane = threadIdx.x & 63;
    const uint64_t wave = wave0 + (threadIdx.x >> 6);
    const uint64_t* rows = rows_of(a, p);
    const uint32_t* ids = ids_of(a, p);
    const uint32_t H = a.H;
    const bool filter = lb > kShortBatch;
    uint64_t t_items = 0, t_segs = 0, t_wread = 0, t_wupd = 0;
    // light entries, straight from the frontier list
    for (uint64_t b = wave; b * lb < n_list; b += n_waves) {
        const uint64_t e = b * lb + lane;
        bool have = false;
        uint32_t slot = 0, q = 0, v = 0, len = 0;
        uint64_t m = 0;
        if ((uint32_t)lane < lb && e < n_list) {
            row_entry(a, s_nfa, ids[e], &slot, &q, &v);
            m = a.lmask[v] & s_nfa.qlab[q];
            const uint64_t work = m ? rpqd::entry_work(a.row_ptr, a.L, s_nfa.delta, v, q, m) : 0;
            have = work != 0 && work <= H;
            len = have ? (uint32_t)work : 0;
        }
        t_segs += __popcll(__ballot(have)) * (lane == 0);
        expand_segments<K, SEEN>(a, s_nfa, rows, filter, have, (uint32_t)e, slot, q, v, m, 0, len, t_items, t_wread, t_wupd);
    }
    // heavy entries, as slices
    const Desc* desc = desc_of(a, p);
    for (uint64_t b = wave; b * db < n_desc; b += n_waves) {
        const uint64_t di = b * db + lane;
        bool have = false;
        uint32_t ent = 0, slot = 0, q = 0, v = 0, len = 0;
        uint64_t m = 0, beg = 0;
        if ((uint32_t)lane < db && di < n_desc) {
            const Desc d = desc[di];
            ent = d.entry;
            beg = d.beg;
            len = d.len;
            row_entry(a, s_nfa, ids[ent], &slot, &q, &v);
            m = a.lmask[v] & s_nfa.qlab[q];
            have = true;
        }
        t_segs += __popcll(__ballot(have)) * (lane == 0);
        expand_segments<K, SEEN>(a, s_nfa, rows, filter, have, ent, slot, q, v, m, beg, len, t_items, t_wread, t_wupd);
    }
    const uint64_t t[4] = {t_items, t_segs, t_wread, t_wupd};
    add_tallies<4>(a, T_ITEMS, t);
}

// ------------------------------------------------------------------------------------------------
// compaction: the rows touched by the last expansion (or by seeding) become the dense list of
// row ids of the next frontier.  Each wave reads 64 consecutive touch words (one per lane),
// clears them, and places its rows with one counter update (popcount prefix over the wave).
// ------------------------------------------------------------------------------------------------
__global__ __launch_bounds__(kBlock) void k_compact(Args a, int p, uint64_t n_rows, uint32_t level) {
    const int np = p ^ 1;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        // the list and slices of parity p were consumed by the expansion that just ran
        a.counters[C_LIST + p] = 0;
        a.counters[C_DESC + p] = 0;
    }
    // the finalize that follows collects its frontier's sources there
    for (uint64_t i = (uint64_t)blockIdx.x * kBlock + threadIdx.x; i < a.n_active; i += (uint64_t)gridDim.x * kBlock)
        a.active[np * a.n_active + i] = 0;
    const int lane = threadIdx.x & 63;
    const uint64_t n_waves = (uint64_t)gridDim.x * kWaves;
    const uint64_t wave = (uint64_t)blockIdx.x * kWaves + (threadIdx.x >> 6);
    const uint64_t n_words = (n_rows + 63) / 64;
    unsigned long long* lcnt = &a.counters[C_LIST + np];
    uint32_t* ids = ids_of(a, np);
    bool appended = false;
    for (uint64_t w0 = wave * 64; w0 < n_words; w0 += n_waves * 64) {
        const uint64_t wi = w0 + lane;
        uint64_t tw = wi < n_words ? a.touch[wi] : 0;
        if (tw) {
            a.touch[wi] = 0;
            if (a.seen_or) {
                const uint64_t ev = a.ever[wi];
                if (tw & ~ev) a.ever[wi] = ev | tw;
                a.fresh[wi] = tw & ~ev;
            }
        }
        const uint32_t c = (uint32_t)__popcll(tw);
        const uint32_t incl = rpqd::wave_incl_scan_u32(c);
        const uint32_t tot = __shfl(incl, 63, 64);
        if (tot == 0) continue;
        appended = true;
        unsigned long long base = 0;
        if (lane == 0) base = atomicAdd(lcnt, (unsigned long long)tot);
        base = __shfl(base, 0, 64);
        uint64_t pos = base + incl - c;
        while (tw) {
            const int b = __ffsll((long long)tw) - 1;
            tw &= tw - 1;
            if (pos < a.list_cap) ids[pos] = (uint32_t)(wi * 64 + b);
            else atomicOr(&a.counters[C_ERR], (unsigned long long)ERR_LIST);
            ++pos;
        }
    }
    if (lane == 0 && appended) atomicMax(&a.counters[C_LASTLEVEL], (unsigned long long)level + 1);
}

// ------------------------------------------------------------------------------------------------
// finalize.  (Seen OR) a row is full when it holds every source of its unit that had a bit in the previous
// frontier: a source without one has ended its search, so nothing can be added to the row any more.  That
// set only shrinks from level to level and a row only grows, so a full row stays full.  Per batch of 64 new
// frontier rows:
//   word phase  groups of K lanes take a row each (lane k, word k): Next moves into the compact
//               frontier row, Vis takes the new bits, and the group counts the new source bits of
//               the row;
//   row phase   lane i takes row i: counts the items of its item space (the product edges each of
//               its new source bits will examine); the slices of rows with more than H items are
//               written by the whole wave.  With count_work == 0 (the last depth of a
//               length-bounded search) the rows are recorded but not prepared for expansion.
// ------------------------------------------------------------------------------------------------
constexpr uint64_t kTrackWords = 1ull << 20;

template <int K, bool SEEN>
__global__ __launch_bounds__(kBlock) void k_finalize(Args a, int p, int count_work) {
    constexpr int GS = 64 / K;
    __shared__ LdsNfa s_nfa;
    const int np = p ^ 1;
    const uint64_t n = min((uint64_t)a.counters[C_LIST + np], a.list_cap);
    const uint64_t n_waves = (uint64_t)gridDim.x * kWaves, wave0 = (uint64_t)blockIdx.x * kWaves;
    const uint32_t fb = batch_of(n, n_waves);
    const uint64_t* was_active = a.active + p * a.n_active;
    unsigned long long* now_active = reinterpret_cast<unsigned long long*>(a.active + np * a.n_active);
    // sources with a bit in the new frontier: word k of slot acc_slot, collected while the wave's rows
    // share a slot.  A stale copy of the word only costs an OR that is not needed.  A short list keeps the
    // previous frontier's sources, which hold its own: every wave's OR of a few words would be most of its
    // time (one source of R-MAT 18: 14 us a launch).  The last block copies them, which has no entries then.
    const bool track = SEEN && n * K >= kTrackWords;
    if (SEEN && !track && blockIdx.x == gridDim.x - 1)
        for (uint64_t i = threadIdx.x; i < a.n_active; i += kBlock) now_active[i] = was_active[i];
    if (wave0 * fb >= n) return;
    const bool mark = fb > kShortBatch;
    load_nfa(a, s_nfa);
    const int lane = threadIdx.x & 63;
    const int grp = lane / K, k = lane % K;
    const uint32_t* ids = ids_of(a, np);
    uint64_t* rows = rows_of(a, np);
    Desc* dout = desc_of(a, np);
    unsigned long long* dcnt = &a.counters[C_DESC + np];
    const uint32_t H = a.H;
    uint64_t eprod = 0, t_rows = 0, t_words = 0, t_fresh = 0;
    const uint64_t gmask = (K == 64) ? ~0ull : (((1ull << (K & 63)) - 1) << (grp * K));
    uint64_t acc_k = 0;
    uint32_t acc_slot = kNone;
    auto put_active = [&](uint32_t sl, uint64_t x) {
        unsigned long long* w = &now_active[(uint64_t)sl * K + k];
        if (x & ~*w) atomicOr(w, (unsigned long long)x);
    };
    auto flush_active = [&]() {
        if (acc_slot == kNone) return;
#pragma unroll
        for (int o = K; o < 64; o <<= 1) acc_k |= __shfl_xor(acc_k, o, 64);
        if (lane < K) put_active(acc_slot, acc_k);
        acc_k = 0;
    };
    const uint64_t wave = wave0 + (threadIdx.x >> 6);
    for (uint64_t e0 = wave * fb; e0 < n; e0 += n_waves * fb) {
        const uint64_t e = e0 + lane;
        const bool active = (uint32_t)lane < fb && e < n;
        const uint32_t my_row = active ? ids[e] : 0;
        uint32_t slot = 0, q = 0, v = 0;
        if (active) row_entry(a, s_nfa, my_row, &slot, &q, &v);
        // seen OR: a row listed for the first time has nothing in the second bitmap yet, which is then
        // written whole and not read: it is not cleared for a group
        const uint64_t fresh = SEEN ? __ballot(active && ((a.fresh[my_row >> 6] >> (my_row & 63)) & 1)) : 0;
        const uint32_t n_here = (uint32_t)min<uint64_t>(fb, n - e0);
        t_rows += n_here * (lane == 0);
        t_fresh += __popcll(fresh) * (lane == 0);
        const uint32_t slot0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)slot);
        const bool one_slot = __ballot(active && slot != slot0) == 0;
        if (SEEN && track && (!one_slot || slot0 != acc_slot)) {
            flush_active();
            acc_slot = one_slot ? slot0 : kNone;
        }
        // a row's items (the product edges of each new source bit): its accesses beside the word phase's.  At
        // the depth bound of a length-bounded query the entries are recorded but never expanded: no product
        // edges, no slices.
        uint64_t work = 0;
        if (active && count_work) {
            const uint64_t m = a.lmask[v] & s_nfa.qlab[q];
            work = m ? rpqd::entry_work(a.row_ptr, a.L, s_nfa.delta, v, q, m) : 0;
        }
        uint32_t my_pc = 0;
        // word phase
        auto words = [&](auto rows_each, uint32_t j) {
            constexpr int U = decltype(rows_each)::value;
            uint32_t r[U], sl[U];
            uint64_t nk[U], ov[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const uint32_t idx = j + u * GS + grp;
                r[u] = __shfl(my_row, idx & 63, 64);
                sl[u] = one_slot ? slot0 : __shfl(slot, idx & 63, 64);
                nk[u] = ov[u] = 0;
                if (idx < n_here) {
                    if constexpr (SEEN) {
                        if (!((fresh >> idx) & 1)) ov[u] = a.next[(uint64_t)r[u] * K + k];
                        nk[u] = a.vis[(uint64_t)r[u] * K + k];
                    } else {
                        nk[u] = a.next[(uint64_t)r[u] * K + k];
                    }
                }
            }
            if constexpr (SEEN) {
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const uint32_t idx = j + u * GS + grp;
                    const bool ok = mark && idx < n_here && (was_active[(uint64_t)sl[u] * K + k] & ~nk[u]) == 0;
                    nk[u] &= ~ov[u];
                    if (one_slot) acc_k |= nk[u];
                    else if (track && idx < n_here && nk[u]) put_active(sl[u], nk[u]);
                    // the row is on the list once: nothing else writes its byte
                    if (mark && (__ballot(ok) & gmask) == gmask && k == 0) a.full[r[u]] = 1;
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const uint32_t idx = j + u * GS + grp;
                uint32_t pc = 0;
                if (idx < n_here) {
                    rows[(e0 + idx) * K + k] = nk[u];
                    // seen OR: the snapshot catches up with Vis.  Two reads: Next is cleared.
                    if (nk[u] || ((fresh >> idx) & 1)) a.next[(uint64_t)r[u] * K + k] = SEEN ? (ov[u] | nk[u]) : 0;
                    if (nk[u]) {
                        // a row is on the list once, and nothing else writes its Vis word in this
                        // kernel: a plain read-modify-write (an atomic OR cost 0.82 vs 0.69 ms a
                        // launch).  With seen OR the expansion has already set these bits.
                        if (!SEEN) a.vis[(uint64_t)r[u] * K + k] |= nk[u];
                        ++t_words;
                        pc = (uint32_t)__popcll(nk[u]);
                    }
                }
#pragma unroll
                for (int o = K / 2; o >= 1; o >>= 1) pc += __shfl_xor(pc, o, 64);
                // lane i keeps the count of row i
                const uint32_t rel = (uint32_t)lane - (j + u * GS);
                const uint32_t got = __shfl(pc, (rel % GS) * K, 64);
                if (rel < (uint32_t)GS) my_pc = got;
            }
        };
        if (SEEN && n_here <= (uint32_t)GS) words(std::integral_constant<int, SEEN ? 1 : kUnroll>(), 0);
        else
            for (uint32_t j = 0; j < n_here; j += GS * kUnroll) words(std::integral_constant<int, kUnroll>(), j);
        // row phase: product edges; entries of more than H items are cut into slices
        eprod += (uint64_t)my_pc * work;
        const uint64_t ndesc = work > H ? (work + H - 1) / H : 0;
        const uint64_t dincl = rpqd::wave_incl_scan_u64(ndesc);
        const uint64_t dexcl = dincl - ndesc;
        const uint64_t dtot = __shfl(dincl, 63, 64);
        if (dtot) {
            unsigned long long dbase = 0;
            if (lane == 0) dbase = atomicAdd(dcnt, (unsigned long long)dtot);
            dbase = __shfl(dbase, 0, 64);
            // the wave writes its slices together: slice i is described by the lane owning it
            for (uint64_t i0 = 0; i0 < dtot; i0 += 64) {
                const uint64_t i = i0 + lane;
                int c = 0;
#pragma unroll
                for (int step = 32; step >= 1; step >>= 1) {
                    const int cand = c + step;
                    const uint64_t ex = __shfl(dexcl, cand, 64);
                    if (ex <= i) c = cand;
                }
                const uint64_t c_work = __shfl(work, c, 64);
                const uint64_t c_ex = __shfl(dexcl, c, 64);
                if (i < dtot) {
                    const uint64_t pos = dbase + i;
                    if (pos < a.desc_cap) {
                        const uint64_t k = i - c_ex;
                        Desc dd;
                        dd.entry = (uint32_t)(e0 + c);
                        dd.beg = k * H;
                        dd.len = (uint32_t)min<uint64_t>(H, c_work - k * H);
                        dout[pos] = dd;
                    } else {
                        atomicOr(&a.counters[C_ERR], (unsigned long long)ERR_DESC);
                    }
                }
            }
        }
    }
    flush_active();
    const uint64_t t[4] = {eprod, t_rows, t_words, t_fresh};
    add_tallies<4>(a, T_EPROD, t);
}

// ------------------------------------------------------------------------------------------------
// sources: validity, which of them get a bit, and the results of those that do not
// ------------------------------------------------------------------------------------------------
constexpr uint32_t kSrcTile = 2048;   // sources per block

struct SrcArgs {
    const uint32_t* sources;   // the caller's list, or null: 0, 1, ...
    uint64_t n;
    const uint64_t* lmask;
    uint64_t init_labels;      // labels that an initial state can follow
    uint32_t V;
    uint32_t compact;          // sources without such a label get no bit
    uint32_t eps;              // the empty word is in the language: (s, s) is a result
    const uint64_t* target;
    uint64_t* per_source;      // [n][2] or null
    unsigned long long* bits;  // [V / 64], zero on entry: sources with a bit, or null if no class needs them
    uint32_t* tile_n;          // sources with a bit per tile
    uint32_t* out_srcs;        // compact: their list and positions
    uint32_t* out_pos;
    unsigned long long* counters;
};

__device__ __forceinline__ bool has_bit(const SrcArgs& a, uint32_t s) {
    return s < a.V && (!a.compact || (a.lmask[s] & a.init_labels));
}

// the zero-length walk of s counts
__device__ __forceinline__ bool self_result(const SrcArgs& a, uint32_t s) {
    return a.eps && (!a.target || ((a.target[s >> 6] >> (s & 63)) & 1));
}

__global__ __launch_bounds__(kBlock) void k_src_count(SrcArgs a) {
    __shared__ uint64_t s_part[kWaves][3];
    const int lane = threadIdx.x & 63;
    uint64_t kept = 0, dead = 0, hash = 0;
    for (uint32_t r = 0; r < kSrcTile; r += kBlock) {
        const uint64_t i = (uint64_t)blockIdx.x * kSrcTile + r + threadIdx.x;
        bool alive = false;
        uint32_t s = 0;
        if (i < a.n) {
            s = a.sources ? a.sources[i] : (uint32_t)i;
            if (a.sources && (s >= a.V || (i > 0 && a.sources[i - 1] >= s)))
                atomicOr(&a.counters[C_ERR], (unsigned long long)ERR_SOURCES);
            alive = has_bit(a, s);
            if (!alive && s < a.V) {
                const bool self = self_result(a, s);
                dead += self;
                hash += self ? rpqd::mix64(((uint64_t)s << 32) | s) : 0;
            }
        }
        const uint64_t m = __ballot(alive);
        kept += (uint64_t)__popcll(m) * (lane == 0);
        if (a.bits && m) {
            // every vertex is a source: the wave's 64 are one word of the bitmap
            if (!a.sources) {
                if (lane == 0) a.bits[i >> 6] = m;
            } else if (alive) {
                atomicOr(&a.bits[s >> 6], 1ull << (s & 63));
            }
        }
    }
    kept = rpqd::wave_sum_u64(kept);
    dead = rpqd::wave_sum_u64(dead);
    hash = rpqd::wave_sum_u64(hash);
    if (lane == 0) {
        s_part[threadIdx.x >> 6][0] = kept;
        s_part[threadIdx.x >> 6][1] = dead;
        s_part[threadIdx.x >> 6][2] = hash;
    }
    __syncthreads();
    if (threadIdx.x < 3) {
        uint64_t t = 0;
        for (int w = 0; w < kWaves; ++w) t += s_part[w][threadIdx.x];
        if (threadIdx.x == 0) a.tile_n[blockIdx.x] = (uint32_t)t;
        else if (t) atomicAdd(&a.counters[threadIdx.x == 1 ? C_COUNT : C_HASH], (unsigned long long)t);
    }
}

// sum of n words over the block, in every thread
__device__ __forceinline__ uint64_t block_sum_of(const uint32_t* x, uint64_t n) {
    __shared__ uint64_t s_sum[kWaves];
    uint64_t t = 0;
    for (uint64_t i = threadIdx.x; i < n; i += kBlock) t += x[i];
    t = rpqd::wave_sum_u64(t);
    if ((threadIdx.x & 63) == 0) s_sum[threadIdx.x >> 6] = t;
    __syncthreads();
    t = 0;
    for (int w = 0; w < kWaves; ++w) t += s_sum[w];
    __syncthreads();
    return t;
}

__global__ __launch_bounds__(kBlock) void k_src_write(SrcArgs a) {
    __shared__ uint32_t s_n[kWaves];
    uint64_t at = block_sum_of(a.tile_n, blockIdx.x);
    if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) a.counters[C_ALIVE] = at + a.tile_n[blockIdx.x];
    const bool valid = a.counters[C_ERR] == 0;   // an invalid call leaves its outputs as they are
    for (uint32_t r = 0; r < kSrcTile; r += kBlock) {
        const uint64_t i = (uint64_t)blockIdx.x * kSrcTile + r + threadIdx.x;
        uint32_t s = 0;
        bool alive = false;
        if (i < a.n) {
            s = a.sources ? a.sources[i] : (uint32_t)i;
            alive = has_bit(a, s);
        }
        const uint64_t m = __ballot(alive);
        if ((threadIdx.x & 63) == 0) s_n[threadIdx.x >> 6] = (uint32_t)__popcll(m);
        __syncthreads();
        uint32_t before = 0, all = 0;
        for (int w = 0; w < kWaves; ++w) {
            before += w < (int)(threadIdx.x >> 6) ? s_n[w] : 0;
            all += s_n[w];
        }
        if (alive) {
            const uint64_t j = at + before + __popcll(m & rpqd::lanemask_lt());
            a.out_srcs[j] = s;
            a.out_pos[j] = (uint32_t)i;
        } else if (valid && a.per_source && i < a.n) {
            const bool self = self_result(a, s);
            a.per_source[2 * i] = self;
            a.per_source[2 * i + 1] = self ? rpqd::mix64(((uint64_t)s << 32) | s) : 0;
        }
        at += all;
        __syncthreads();
    }
}

// ------------------------------------------------------------------------------------------------
// bit order.  A word of a row is expanded once for every level at which one of its 64 sources arrives, so
// sources that arrive together belong into one word.  Two sources with an edge to the same hub are at most
// two levels apart at every vertex, and mostly not apart at all; so a group's sources are ordered by the
// largest degree among (up to kScoreEdges of) their first neighbours, and within it by that neighbour.
// One counting pass over kScores buckets; the order within a bucket is of no consequence.
// ------------------------------------------------------------------------------------------------
constexpr uint32_t kScoreEdges = 16;
constexpr uint32_t kScores = 1u << 16;   // 5 bits of degree, 8 of the neighbour, 3 that spread a hub's counter

struct OrderArgs {
    const uint32_t* row_ptr;
    const uint32_t* dst;
    const uint64_t* lmask;
    uint64_t init_labels;
    uint32_t L;
    uint64_t n, gbase;           // the group
    const uint32_t* in_srcs;     // ascending
    const uint32_t* in_pos;
    uint64_t* hist;              // [kScores]: zero, then counts, then their prefixes
    uint32_t* score;             // [n]
    uint32_t* rank;              // [n]
    uint32_t* srcs;
    uint32_t* pos;
    uint32_t* bit_of;
};

__global__ __launch_bounds__(kBlock) void k_order_score(OrderArgs a) {
    const uint64_t i = (uint64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i >= a.n) return;
    const uint32_t s = a.in_srcs[a.gbase + i];
    uint32_t best = 0, hub = 0;
    for (uint64_t m = a.lmask[s] & a.init_labels; m; m &= m - 1) {
        const uint64_t r = (uint64_t)s * a.L + (uint32_t)(__ffsll((long long)m) - 1);
        const uint32_t b = a.row_ptr[r], d = a.row_ptr[r + 1] - b;
        const uint32_t n = min(d, kScoreEdges);
        for (uint32_t t = 0; t < n; ++t) {
            const uint32_t w = a.dst[b + (uint32_t)((uint64_t)d * t / n)];
            const uint64_t rw = (uint64_t)w * a.L;
            const uint32_t deg = a.row_ptr[rw + a.L] - a.row_ptr[rw];
            if (deg > best || (deg == best && w > hub)) {
                best = deg;
                hub = w;
            }
        }
    }
    const uint32_t bits = best ? 32 - __clz(best) : 0;
    const uint32_t score = ((31 - min(bits, 31u)) << 11) | (((hub * 0x9E3779B1u) >> 24) << 3) | (threadIdx.x & 7);
    a.score[i] = score;
    a.rank[i] = (uint32_t)atomicAdd(reinterpret_cast<unsigned long long*>(&a.hist[score]), 1ull);
}

__global__ __launch_bounds__(kBlock) void k_order_place(OrderArgs a) {
    const uint64_t i = (uint64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i >= a.n) return;
    const uint32_t bit = (uint32_t)a.hist[a.score[i]] + a.rank[i];
    a.srcs[a.gbase + bit] = a.in_srcs[a.gbase + i];
    a.pos[a.gbase + bit] = a.in_pos[a.gbase + i];
    a.bit_of[a.gbase + i] = bit;
}

// ------------------------------------------------------------------------------------------------
// classes: the vertices a set of labels can lead to (and, if asked, the sources), as a rank table and
// an ascending list.  One wave per 64 words of vertex bits; a first pass counts, a second sums the counts
// before it and writes.
// ------------------------------------------------------------------------------------------------
constexpr int kMaxClasses = RPQ_MAX_STATES + 2;

struct ClassArgs {
    uint64_t labels[kMaxClasses];
    uint64_t list_at[kMaxClasses];
    uint64_t src;                 // bit c: class c holds the sources too
    const uint64_t* entered;      // [L][n_words]
    const unsigned long long* src_bits;
    uint64_t n_words;
    uint32_t n_tiles;             // of 64 words
    uint32_t* tile_n;             // [classes][n_tiles]
    ulonglong2* rank;             // [classes][n_words]
    uint32_t* verts;
    uint32_t* class_n;            // [classes]
};

__device__ __forceinline__ uint64_t class_word(const ClassArgs& a, uint32_t c, uint64_t w) {
    uint64_t x = (a.src >> c) & 1 ? a.src_bits[w] : 0;
    for (uint64_t m = a.labels[c]; m; m &= m - 1) x |= a.entered[(uint64_t)(__ffsll((long long)m) - 1) * a.n_words + w];
    return x;
}

__global__ __launch_bounds__(kBlock) void k_class_count(ClassArgs a) {
    const uint32_t c = blockIdx.y, tile = blockIdx.x * kWaves + (threadIdx.x >> 6);
    if (tile >= a.n_tiles) return;
    const uint64_t w = (uint64_t)tile * 64 + (threadIdx.x & 63);
    const uint64_t t = rpqd::wave_sum_u64(w < a.n_words ? (uint64_t)__popcll(class_word(a, c, w)) : 0);
    if ((threadIdx.x & 63) == 0) a.tile_n[(uint64_t)c * a.n_tiles + tile] = (uint32_t)t;
}

__global__ __launch_bounds__(kBlock) void k_class_write(ClassArgs a) {
    const uint32_t c = blockIdx.y, tile0 = blockIdx.x * kWaves, tile = tile0 + (threadIdx.x >> 6);
    const uint32_t* tn = a.tile_n + (uint64_t)c * a.n_tiles;
    uint64_t at = block_sum_of(tn, tile0);
    for (uint32_t t = tile0; t < tile && t < a.n_tiles; ++t) at += tn[t];
    if (tile >= a.n_tiles) return;
    const int lane = threadIdx.x & 63;
    const uint64_t w = (uint64_t)tile * 64 + lane;
    const uint64_t x = w < a.n_words ? class_word(a, c, w) : 0;
    const uint32_t n = (uint32_t)__popcll(x);
    const uint32_t incl = rpqd::wave_incl_scan_u32(n);
    const uint64_t before = at + incl - n;
    if (w < a.n_words) a.rank[(uint64_t)c * a.n_words + w] = make_ulonglong2(x, before);
    if (tile == a.n_tiles - 1 && lane == 63) a.class_n[c] = (uint32_t)(at + incl);
    uint32_t* verts = a.verts + a.list_at[c];
    for (int j = 0; j < 64; ++j) {
        const uint64_t xj = __shfl(x, j, 64), bj = __shfl(before, j, 64);
        if ((xj >> lane) & 1) verts[bj + __popcll(xj & rpqd::lanemask_lt())] = (uint32_t)((w - lane + j) * 64 + lane);
    }
}

// ------------------------------------------------------------------------------------------------
// seeding: (q0, s_i) for every initial state q0 and every source of the group
// ------------------------------------------------------------------------------------------------
__global__ __launch_bounds__(kBlock) void k_seed(Args a, uint32_t G, uint32_t K) {
    const uint64_t i = (uint64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i == 0) {
        // a new group: no list or slice is left (a length-bounded group ends with a frontier), no level ran
        a.counters[C_LIST] = a.counters[C_LIST + 1] = a.counters[C_DESC] = a.counters[C_DESC + 1] = 0;
        a.counters[C_LASTLEVEL] = 0;
    }
    if (i >= (uint64_t)G * a.W) return;
    const uint64_t gi = a.gbase + i;
    // before the first frontier every source of the unit counts as searching
    if ((i & 63) == 0) {
        const uint64_t n = gi < a.n_srcs ? a.n_srcs - gi : 0;
        a.active[i >> 6] = n >= 64 ? ~0ull : (1ull << n) - 1;
    }
    if (gi >= a.n_srcs) return;
    const uint32_t slot = (uint32_t)(i / a.W), j = (uint32_t)(i % a.W);
    const uint32_t s = a.srcs ? a.srcs[gi] : (uint32_t)gi;
    const uint32_t k = j >> 6;
    const uint64_t bit = 1ull << (j & 63);
    uint32_t init = a.nfa->init;
    while (init) {
        const uint32_t q = __ffs(init) - 1;
        init &= init - 1;
        const uint32_t kind = a.nfa->kind[q];
        const uint32_t off = kind == ROW_SOURCE ? j : kind == ROW_ALL ? s : rank_in(a.rank, a.nfa->rank_at[q], s);
        const uint64_t row = (uint64_t)slot * a.R + a.nfa->base[q] + off;
        or_relaxed(&(a.seen_or ? a.vis : a.next)[row * K + k], bit);
        or_relaxed(&a.touch[row >> 6], 1ull << (row & 63));
    }
}

// ------------------------------------------------------------------------------------------------
// The whole search of a small graph.  Sources do not meet each other's bits, so a block takes 32 of them
// from the seeds to the fixpoint by itself, with a word of visited and a word of Next bits per row in LDS,
// and writes its half words of the visited bitmap once: no list, no launch and no wait of the host per
// level.  A level is a chain of dependent LDS and cache accesses between two barriers, 3.2 us (4.1 with the
// frontier gathered from LDS and only four edges of a row by its own lane; fewer sources a block, or the
// adjacency in LDS too, gained nothing); three launches and a quarter of a wait take 27.  1,000 vertices,
// 5,000 edges, all pairs with keys in 40 levels: 1.30 -> 0.25 ms a call.
// A listed row's Next word holds its frontier bits (they are in Vis) and the bits found at this level
// (they are not), so two words a row do.
// ------------------------------------------------------------------------------------------------
constexpr uint32_t kSmallRows = 16384;         // two words each: 128 of the 160 KB of LDS
// items of a level, which one block visits alone.  4,000 vertices, 400,000 edges, 3 states (1.2 M items):
// 64 sources 0.40 ms against 0.49 by levels, one source 0.23 against 0.30; the gap closes from there on
constexpr uint64_t kSmallItems = 1ull << 20;
constexpr int kSmallBlock = 1024;
constexpr int kOwn = 4;   // edges in flight a lane
constexpr int kSmallWaves = kSmallBlock / 64;

__global__ __launch_bounds__(kSmallBlock) void k_small_search(Args a, uint64_t max_len) {
    extern __shared__ uint32_t s_rows[];
    __shared__ uint32_t s_delta[RPQ_MAX_STATES * RPQ_MAX_LABELS];
    __shared__ uint64_t s_qlab[RPQ_MAX_STATES];
    __shared__ uint32_t s_base[RPQ_MAX_STATES];
    __shared__ uint16_t s_queue[kSmallWaves][128];   // a wave's frontier rows
    __shared__ uint64_t s_part[kSmallWaves];
    const uint32_t R = a.R, tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    uint32_t* const s_vis = s_rows;
    uint32_t* const s_next = s_rows + R;
    for (uint32_t i = tid; i < a.Q * a.L; i += kSmallBlock) s_delta[i] = a.nfa->delta[i];
    if (tid < a.Q) {
        s_qlab[tid] = a.nfa->qlab[tid];
        s_base[tid] = a.nfa->base[tid];
    }
    for (uint32_t r = tid; r < 2 * R; r += kSmallBlock) s_rows[r] = 0;
    __syncthreads();
    const uint64_t gi = (uint64_t)blockIdx.x * 32 + tid;
    if (tid < 32 && gi < a.n_srcs) {
        const uint32_t v = a.srcs ? a.srcs[gi] : (uint32_t)gi;
        for (uint32_t f = a.nfa->init; f; f &= f - 1) atomicOr(&s_next[s_base[__ffs(f) - 1] + v], 1u << tid);
    }
    __syncthreads();
    uint16_t* const queue = s_queue[wave];
    uint32_t top = 1;
    while (2 * top < a.Q) top *= 2;
    auto visit = [&](uint32_t w, uint32_t bits, uint32_t to) {
        for (; to; to &= to - 1) {
            const uint32_t t = s_base[__ffs(to) - 1] + w;
            const uint32_t n = bits & ~s_vis[t];
            if (n) atomicOr(&s_next[t], n);
        }
    };
    uint64_t eprod = 0, level = 0;
    // every level with a frontier sets a bit of Vis, so the loop ends
    for (;; ++level) {
        // bit i: the thread's i-th row is on the frontier
        uint32_t hot = 0;
        for (uint32_t i0 = 0; i0 * kSmallBlock < R; i0 += 4) {
            uint32_t v[4], n[4];
#pragma unroll
            for (uint32_t u = 0; u < 4; ++u) {
                const uint32_t r = (i0 + u) * kSmallBlock + tid;
                v[u] = r < R ? s_vis[r] : 0;
                n[u] = r < R ? s_next[r] : 0;
            }
#pragma unroll
            for (uint32_t u = 0; u < 4; ++u) {
                const uint32_t r = (i0 + u) * kSmallBlock + tid;
                n[u] &= ~v[u];
                if (r < R) {
                    s_next[r] = n[u];
                    s_vis[r] = v[u] | n[u];
                }
                hot |= (uint32_t)(n[u] != 0) << (i0 + u);
            }
        }
        if (!__syncthreads_or((int)hot)) break;
        if (level >= max_len) {   // recorded, not expanded
            ++level;
            break;
        }
        uint32_t queued = 0;   // wave-uniform
        for (uint32_t i = 0; i * kSmallBlock < R || queued; ++i) {
            const bool on = i * kSmallBlock < R && ((hot >> i) & 1);
            const uint64_t m = __ballot(on);
            if (on) queue[queued + __popcll(m & rpqd::lanemask_lt())] = (uint16_t)(i * kSmallBlock + tid);
            queued += (uint32_t)__popcll(m);
            if (queued == 0 || (queued < 64 && (i + 1) * kSmallBlock < R)) continue;
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            const uint32_t take = min(queued, 64u);
            uint2 row = make_uint2(0, 0);   // its number and its frontier bits
            if ((uint32_t)lane < take) {
                row.x = queue[lane];
                row.y = __hip_atomic_load(&s_next[row.x], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) & s_vis[row.x];
            }
            const uint16_t rest = queue[64 + lane];
            queued -= take;
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            if ((uint32_t)lane < queued) queue[lane] = rest;
            uint32_t q = 0;   // the last state whose rows begin at or before the row
            for (uint32_t step = top; step >= 1; step >>= 1)
                if (q + step < a.Q && s_base[q + step] <= row.x) q += step;
            const uint64_t at = (uint64_t)(row.x - s_base[q]) * a.L;
            uint64_t labels = row.y ? s_qlab[q] : 0;
            while (__ballot(labels != 0)) {
                uint32_t lo = 0, deg = 0, to = 0;
                if (labels) {
                    const int l = __ffsll((long long)labels) - 1;
                    labels &= labels - 1;
                    lo = a.row_ptr[at + l];
                    deg = a.row_ptr[at + l + 1] - lo;
                    to = s_delta[q * a.L + l];
                    eprod += (uint64_t)__popc(row.y) * __popc(to) * deg;
                }
                // a row's first edges by its own lane, the others spread over the wave
                uint32_t w[kOwn];
                for (int turn = 0; turn < 2 && __ballot(deg != 0); ++turn) {
#pragma unroll
                    for (int u = 0; u < kOwn; ++u) w[u] = (uint32_t)u < deg ? a.dst[lo + u] : 0;
#pragma unroll
                    for (int u = 0; u < kOwn; ++u) visit(w[u], row.y, (uint32_t)u < deg ? to : 0);
                    lo += kOwn;
                    deg = deg > kOwn ? deg - kOwn : 0;
                }
                if (__ballot(deg != 0) == 0) continue;
                const uint32_t incl = rpqd::wave_incl_scan_u32(deg), excl = incl - deg;
                const uint32_t total = __shfl(incl, 63, 64);
                for (uint32_t i0 = 0; i0 < total; i0 += 64 * kOwn) {
                    uint32_t c[kOwn];
#pragma unroll
                    for (int u = 0; u < kOwn; ++u) {
                        const uint32_t i = i0 + u * 64 + lane;
                        c[u] = 0;   // the last lane whose edges begin at or before item i
#pragma unroll
                        for (int step = 32; step >= 1; step >>= 1)
                            if ((uint32_t)__shfl(excl, c[u] + step, 64) <= i) c[u] += step;
                        const uint32_t e = (uint32_t)__shfl(lo - excl, c[u], 64) + i;
                        w[u] = i < total ? a.dst[e] : 0;
                    }
#pragma unroll
                    for (int u = 0; u < kOwn; ++u) {
                        const uint32_t bits_of = __shfl(row.y, c[u], 64), to_of = __shfl(to, c[u], 64);
                        visit(w[u], bits_of, i0 + u * 64 + lane < total ? to_of : 0);
                    }
                }
            }
        }
        __syncthreads();
    }
    // the half words of these sources, zero beyond the last
    const uint32_t slot = blockIdx.x * 32 / a.W, half = blockIdx.x * 32 % a.W / 32, halves = a.W / 32;
    uint32_t* const vis = reinterpret_cast<uint32_t*>(a.vis) + (uint64_t)slot * R * halves + half;
    for (uint32_t r = tid; r < R; r += kSmallBlock) vis[(uint64_t)r * halves] = s_vis[r];
    eprod = rpqd::wave_sum_u64(eprod);
    if (lane == 0) s_part[wave] = eprod;
    __syncthreads();
    if (tid == 0) {
        eprod = 0;
        for (int w = 0; w < kSmallWaves; ++w) eprod += s_part[w];
        a.tally[(uint64_t)blockIdx.x * kTallyStride + T_EPROD] += eprod;
        atomicMax(&a.counters[C_LASTLEVEL], (unsigned long long)level);   // levels with a frontier
    }
}

// ------------------------------------------------------------------------------------------------
// extraction
// ------------------------------------------------------------------------------------------------
// Answer words each lane loads per vertex: four adjacent words (two 16-byte loads) where K allows.
// Neighbouring lanes read rows one row (K words) apart, so every lane makes its own memory request;
// loading four words per request instead of one cuts the requests per byte fourfold.
template <int K>
constexpr int kExtractWords() { return K >= 4 ? 4 : (K >= 2 ? 2 : 1); }

enum ExtractMode { X_TOTALS = 0, X_TALLIES = 1, X_KEYS = 2 };

struct ExtractArgs {
    uint32_t G, nchunks, chunk;    // units; chunks of answer vertices
    unsigned long long* acc;       // [G * W][2] count and checksum (tallies)
    uint32_t* partial;             // [G * W][nchunks] keys per chunk (tallies), their prefixes (keys), or null
    const uint64_t* srcbase;       // [G * W] first key of each source (keys)
    uint64_t* pairs;
    uint64_t off, cap;             // keys [off, off + cap) are written
};

__device__ __forceinline__ uint64_t wave_or_u64(uint64_t v) {
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) v |= __shfl_xor(v, o, 64);
    return v;
}

// One wave per (slot, block of kExtractWords consecutive words, chunk of answer vertices).  Lane i loads
// answer vertex i's words: the OR of its rows of final states.  A word block of 64 vertices x 64 sources
// is then walked by rows or by columns, whichever takes fewer steps for what it holds:
//   rows     for each vertex with a bit, lane i is source i: checksums are one lane-constant mix per pair,
//            bound by its five multiplications where the block is dense (41 G pairs in 30.6 ms);
//   columns  for each source with a bit, lane i is vertex i: a source's keys are written as one run (64
//            streams of single keys wrote 4.6 times the bytes: 87 M keys 1.10 -> 0.45 ms), and a few
//            sources do not cost a step per vertex.
// The totals of a call that asks for neither keys nor per-source results need no accumulator per source.
template <int K, int MODE>
__global__ __launch_bounds__(kBlock) void k_extract(Args a, ExtractArgs x) {
    constexpr int KP = kExtractWords<K>();
    constexpr int NKP = K / KP;
    const int lane = threadIdx.x & 63;
    const uint64_t n_waves = (uint64_t)gridDim.x * kWaves;
    const uint64_t total = (uint64_t)x.G * NKP * x.nchunks;
    const DevNfa& nfa = *a.nfa;
    const bool all = nfa.ans_class == kNone;
    const uint32_t n_ans = all ? a.V : a.class_n[nfa.ans_class];
    const uint32_t finals = nfa.final, W = a.W;
    const int wave = threadIdx.x >> 6;
    __shared__ uint32_t s_cnt[MODE == X_TALLIES ? kWaves : 1][64];
    __shared__ uint64_t s_hash[MODE == X_TALLIES ? kWaves : 1][64];
    uint64_t tot_c = 0, tot_h = 0;
    for (uint64_t wv0 = (uint64_t)blockIdx.x * kWaves; wv0 < total; wv0 += n_waves) {
        const uint64_t wv = wv0 + wave;
        // a block's waves that share their sources add up before the sums leave it: adds to one address take
        // 12 ns each (R-MAT 18, one source: 35 -> 17 us)
        const bool together = MODE == X_TALLIES && wv0 / x.nchunks == (wv0 + kWaves - 1) / x.nchunks;
        if (wv >= total) continue;   // then the waves of its block do not share theirs
        const uint32_t chunk = (uint32_t)(wv % x.nchunks);
        const uint32_t kp = (uint32_t)((wv / x.nchunks) % NKP);
        const uint32_t slot = (uint32_t)(wv / ((uint64_t)x.nchunks * NKP));
        const uint32_t ibeg = min(n_ans, chunk * x.chunk);
        const uint32_t iend = min(n_ans, ibeg + x.chunk);
        const uint64_t* vis = a.vis + (uint64_t)slot * a.R * K + (uint64_t)kp * KP;
        uint32_t src[KP];
        uint32_t cnt[KP];   // at most the chunk's vertices
        uint64_t h[KP], cursor[KP];
        rpqd::MixSource ms[KP];
        bool in_window = MODE != X_KEYS;
#pragma unroll
        for (int u = 0; u < KP; ++u) {
            const uint64_t si = (uint64_t)slot * W + (uint64_t)(kp * KP + u) * 64 + lane;
            const uint64_t gi = a.gbase + si;
            const bool valid = gi < a.n_srcs;
            src[u] = valid ? (a.srcs ? a.srcs[gi] : (uint32_t)gi) : 0;
            ms[u] = rpqd::mix_source(src[u]);
            cnt[u] = 0;
            h[u] = cursor[u] = 0;
            if (MODE == X_KEYS && valid) {
                // this source's keys in this chunk are [cursor, end): partial holds the source's chunk
                // prefixes, acc its total
                const uint32_t* pp = x.partial + si * x.nchunks;
                cursor[u] = x.srcbase[si] + pp[chunk];
                const uint64_t end =
                    x.srcbase[si] + (chunk + 1 < x.nchunks ? (uint64_t)pp[chunk + 1] : x.acc[2 * si]);
                in_window |= end > cursor[u] && end > x.off && cursor[u] < x.off + x.cap;
            }
        }
        // a wave none of whose keys fall in the output window has nothing to write
        if (MODE == X_KEYS && __ballot(in_window) == 0) continue;
        for (uint32_t i0 = ibeg; i0 < iend; i0 += 64) {
            const uint32_t i = i0 + lane;
            uint32_t v = 0;
            uint64_t word[KP];
#pragma unroll
            for (int u = 0; u < KP; ++u) word[u] = 0;
            if (i < iend) {
                v = all ? i : a.verts[nfa.ans_list_at + i];
                for (uint32_t f = finals; f; f &= f - 1) {
                    const uint32_t q = __ffs(f) - 1;
                    uint32_t r = kNone;
                    if (nfa.kind[q] == ROW_ALL) {
                        r = v;
                    } else if (nfa.kind[q] == ROW_RANKED) {
                        if (!all && nfa.rank_at[q] == nfa.ans_rank_at) {
                            r = i;
                        } else {
                            const ulonglong2 e = a.rank[nfa.rank_at[q] + (v >> 6)];
                            if ((e.x >> (v & 63)) & 1)
                                r = (uint32_t)e.y + (uint32_t)__popcll(e.x & ((1ull << (v & 63)) - 1));
                        }
                    }
                    if (r == kNone || nfa.base[q] == nfa.base[q + 1]) continue;
                    const uint64_t* p = vis + (uint64_t)(nfa.base[q] + r) * K;
                    if constexpr (KP >= 2) {
#pragma unroll
                        for (int u = 0; u < KP; u += 2) {
                            const ulonglong2 w2 = *reinterpret_cast<const ulonglong2*>(p + u);
                            word[u] |= w2.x;
                            word[u + 1] |= w2.y;
                        }
                    } else {
                        word[0] |= p[0];
                    }
                }
                if (nfa.src_rank_at != kNone) {
                    // the empty word: v itself, if it is a source of this unit and of this word block
                    const ulonglong2 e = a.rank[nfa.src_rank_at + (v >> 6)];
                    const uint64_t order = (uint64_t)e.y + __popcll(e.x & ((1ull << (v & 63)) - 1));
                    if (((e.x >> (v & 63)) & 1) && order >= a.gbase && order - a.gbase < (uint64_t)x.G * W) {
                        const uint64_t bit = a.bit_of ? a.bit_of[order] : order - a.gbase;
                        const uint64_t j = bit - (uint64_t)slot * W - (uint64_t)kp * KP * 64;
#pragma unroll
                        for (int u = 0; u < KP; ++u)
                            if (j >> 6 == (uint64_t)u) word[u] |= 1ull << (j & 63);
                    }
                }
                if (a.target && !((a.target[v >> 6] >> (v & 63)) & 1)) {
#pragma unroll
                    for (int u = 0; u < KP; ++u) word[u] = 0;
                }
            }
#pragma unroll
            for (int u = 0; u < KP; ++u) {
                uint64_t any = __ballot(word[u] != 0);
                if (any == 0) continue;
                uint64_t cols = wave_or_u64(word[u]);
                const uint32_t nr = (uint32_t)__popcll(any), nc = (uint32_t)__popcll(cols);
                if (MODE == X_KEYS ? nc < 8 * nr : MODE == X_TALLIES ? 5 * nc < 2 * nr : 3 * nc < 2 * nr) {
                    while (cols) {
                        const int c = __ffsll((long long)cols) - 1;
                        cols &= cols - 1;
                        const bool bit = (word[u] >> c) & 1;
                        const uint32_t s = (uint32_t)__builtin_amdgcn_readlane((int)src[u], c);
                        if constexpr (MODE == X_KEYS) {
                            const uint64_t m = __ballot(bit);
                            const uint64_t cur = rpqd::readlane_u64(cursor[u], c);
                            const uint64_t at = cur + __popcll(m & rpqd::lanemask_lt());
                            if (bit && at >= x.off && at - x.off < x.cap) x.pairs[at - x.off] = ((uint64_t)s << 32) | v;
                            if (lane == c) cursor[u] = cur + __popcll(m);
                        } else {
                            const uint64_t hv = bit ? rpqd::mix64(((uint64_t)s << 32) | v) : 0;
                            if constexpr (MODE == X_TOTALS) {
                                cnt[u] += bit;
                                h[u] += hv;
                            } else {
                                const uint64_t hs = rpqd::wave_sum_u64(hv);
                                const uint64_t m = __ballot(bit);
                                if (lane == c) {
                                    cnt[u] += (uint32_t)__popcll(m);
                                    h[u] += hs;
                                }
                            }
                        }
                    }
                } else {
                    uint32_t row_bits = 0;   // wave-uniform
                    while (any) {
                        const int j = __ffsll((long long)any) - 1;
                        any &= any - 1;
                        const uint64_t wj = rpqd::readlane_u64(word[u], j);
                        const uint32_t vj = (uint32_t)__builtin_amdgcn_readlane((int)v, j);
                        // the word itself is the mask of the lanes whose source reaches the vertex
                        if constexpr (MODE == X_TOTALS) row_bits += (uint32_t)__popcll(wj);
                        if (__builtin_amdgcn_inverse_ballot_w64(wj)) {
                            if constexpr (MODE == X_KEYS) {
                                if (cursor[u] >= x.off && cursor[u] - x.off < x.cap)
                                    x.pairs[cursor[u] - x.off] = ((uint64_t)src[u] << 32) | vj;
                                ++cursor[u];
                            } else {
                                if constexpr (MODE == X_TALLIES) ++cnt[u];
                                h[u] += rpqd::mix_pair(ms[u], vj);
                            }
                        }
                    }
                    if constexpr (MODE == X_TOTALS) tot_c += lane == 0 ? row_bits : 0;
                }
            }
        }
        if constexpr (MODE == X_TOTALS) {
#pragma unroll
            for (int u = 0; u < KP; ++u) {
                tot_c += cnt[u];
                tot_h += h[u];
            }
        }
        if constexpr (MODE == X_TALLIES) {
#pragma unroll
            for (int u = 0; u < KP; ++u) {
                const uint64_t si = (uint64_t)slot * W + (uint64_t)(kp * KP + u) * 64 + lane;
                const bool valid = a.gbase + si < a.n_srcs;
                if (x.partial && valid) x.partial[si * x.nchunks + chunk] = cnt[u];
                if (!together) {
                    if (valid && cnt[u]) {
                        atomicAdd(&x.acc[2 * si], (unsigned long long)cnt[u]);
                        atomicAdd(&x.acc[2 * si + 1], (unsigned long long)h[u]);
                    }
                    continue;
                }
                s_cnt[wave][lane] = valid ? cnt[u] : 0;
                s_hash[wave][lane] = h[u];
                __syncthreads();
                if (wave == 0 && valid) {
                    uint64_t c = 0, t = 0;
                    for (int w = 0; w < kWaves; ++w) {
                        c += s_cnt[w][lane];
                        t += s_hash[w][lane];
                    }
                    if (c) {
                        atomicAdd(&x.acc[2 * si], (unsigned long long)c);
                        atomicAdd(&x.acc[2 * si + 1], (unsigned long long)t);
                    }
                }
                __syncthreads();
            }
        }
    }
    if constexpr (MODE == X_TOTALS) {
        __shared__ uint64_t s_part[kWaves][2];
        tot_c = rpqd::wave_sum_u64(tot_c);
        tot_h = rpqd::wave_sum_u64(tot_h);
        if (lane == 0) {
            s_part[threadIdx.x >> 6][0] = tot_c;
            s_part[threadIdx.x >> 6][1] = tot_h;
        }
        __syncthreads();
        if (threadIdx.x < 2) {
            uint64_t t = 0;
            for (int w = 0; w < kWaves; ++w) t += s_part[w][threadIdx.x];
            a.xtally[2 * (uint64_t)blockIdx.x + threadIdx.x] += t;
        }
    }
}

// Exclusive chunk prefixes of each source's keys; one wave per source.
__global__ __launch_bounds__(kBlock) void k_chunk_prefix(uint32_t* __restrict__ partial, uint64_t n, uint32_t nchunks) {
    const int lane = threadIdx.x & 63;
    for (uint64_t i = (uint64_t)blockIdx.x * kWaves + (threadIdx.x >> 6); i < n; i += (uint64_t)gridDim.x * kWaves) {
        uint32_t* pp = partial + i * nchunks;
        uint32_t run = 0;
        for (uint32_t c0 = 0; c0 < nchunks; c0 += 512) {
            uint32_t t[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) t[u] = c0 + u * 64 + lane < nchunks ? pp[c0 + u * 64 + lane] : 0;
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const uint32_t c = c0 + u * 64 + lane;
                if (c0 + u * 64 >= nchunks) break;
                const uint32_t incl = rpqd::wave_incl_scan_u32(t[u]);
                if (c < nchunks) pp[c] = run + incl - t[u];
                run += __shfl(incl, 63, 64);
            }
        }
    }
}

// Per-source results of the group and its totals; with SCAN (one block) also the sources' first keys.
template <bool SCAN>
__global__ __launch_bounds__(1024) void k_group_finish(Args a, const unsigned long long* __restrict__ acc,
                                                       uint64_t* __restrict__ srcbase,
                                                       uint64_t* __restrict__ per_source, uint64_t n_group) {
    __shared__ uint64_t s_w[16];
    __shared__ uint64_t s_h[16];
    __shared__ uint64_t s_carry;
    const int t = threadIdx.x;
    const int lane = t & 63, wv = t >> 6;
    if (SCAN && t == 0) s_carry = a.counters[C_PAIRBASE];
    uint64_t csum = 0, hsum = 0;
    __syncthreads();
    for (uint64_t b0 = (uint64_t)blockIdx.x * 1024; b0 < n_group; b0 += (uint64_t)gridDim.x * 1024) {
        // in ascending order of the sources; j is the source's bit
        const uint64_t i = b0 + t;
        const bool valid = i < n_group && a.gbase + i < a.n_srcs;
        const uint64_t j = valid && a.bit_of ? a.bit_of[a.gbase + i] : i;
        const uint64_t c = valid ? acc[2 * j] : 0;
        const uint64_t h = valid ? acc[2 * j + 1] : 0;
        csum += c;
        hsum += h;
        if (valid && per_source) {
            const uint64_t at = a.pos ? a.pos[a.gbase + j] : a.gbase + j;
            per_source[2 * at] = c;
            per_source[2 * at + 1] = h;
        }
        if (SCAN) {
            const uint64_t incl = rpqd::wave_incl_scan_u64(c);
            if (lane == 63) s_w[wv] = incl;
            __syncthreads();
            uint64_t pre = s_carry;
            for (int w = 0; w < wv; ++w) pre += s_w[w];
            if (valid) srcbase[j] = pre + incl - c;
            __syncthreads();
            if (t == 0) {
                uint64_t tot = 0;
                for (int w = 0; w < 16; ++w) tot += s_w[w];
                s_carry += tot;
            }
            __syncthreads();
        }
    }
    csum = rpqd::wave_sum_u64(csum);
    hsum = rpqd::wave_sum_u64(hsum);
    __syncthreads();
    if (lane == 0) {
        s_w[wv] = csum;
        s_h[wv] = hsum;
    }
    __syncthreads();
    if (t == 0) {
        csum = hsum = 0;
        for (int w = 0; w < 16; ++w) {
            csum += s_w[w];
            hsum += s_h[w];
        }
        atomicAdd(&a.counters[C_COUNT], (unsigned long long)csum);
        atomicAdd(&a.counters[C_HASH], (unsigned long long)hsum);
        if (SCAN) a.counters[C_PAIRBASE] = s_carry;
    }
}

// ------------------------------------------------------------------------------------------------
// host side
// ------------------------------------------------------------------------------------------------
// What a call's rows look like, from the automaton, the direction's entered labels and the number of
// sources: fixed before the sources are looked at.
struct Plan {
    DevNfa dn;                  // base[] is set with the unit width
    const rpq::Csr* csr;
    uint64_t rows[RPQ_MAX_STATES];   // upper bound of a state's rows (ROW_SOURCE: the unit width instead)
    uint32_t n_classes;
    uint64_t labels[kMaxClasses];
    uint64_t bound[kMaxClasses];     // upper bound of a class's vertices
    uint64_t list_at[kMaxClasses];
    uint64_t src;                    // bit c: class c holds the sources
    uint64_t verts;                  // vertices over all classes
    uint64_t ans_bound;              // answer vertices
    uint64_t init_labels;
    bool eps, compact_src;
    uint64_t n_words, desc_items;    // words of V bits; items of a level and unit, at most
};

struct Layout {
    uint32_t K, W, G, Q, L, V, H, R, nchunks, chunk, sync_every;
    bool order;         // sources are ordered within their group
    uint32_t seen_or;   // visit scheme of the expansion (1 = seen OR, 0 = two reads)
    uint64_t max_len;   // deepest level finalized: the length bound, or no bound (UINT64_MAX)
    uint64_t list_cap, desc_cap;
    // fixed by the plan and the number of sources
    uint64_t off_counters, off_tally, off_xtally, off_src_bits, zero_words, off_nfa, off_tile_n, off_srcs, off_pos,
        off_srcs2, off_pos2, off_bit_of, off_hist, off_score, off_rank, off_verts, off_class_n, off_class_tile_n;
    // by the unit width and units in flight
    uint64_t off_vis, off_next, off_vis2, off_touch, off_ever, off_fresh, off_full, off_active, off_ids[2],
        off_rows[2], off_desc[2], off_acc, off_partial, off_srcbase, total;
};

uint64_t align256(uint64_t x) { return (x + 255) & ~255ull; }

int popc64(uint64_t x) { return __builtin_popcountll(x); }

int validate_nfa(const rpq_graph* g, const rpq_nfa* nfa) {
    if (!nfa) {
        rpq::set_error("automaton is NULL");
        return RPQ_EINVAL;
    }
    if (nfa->n_states == 0 || nfa->n_states > RPQ_MAX_STATES) {
        rpq::set_error("automaton has %u states; 1..%d supported", nfa->n_states, RPQ_MAX_STATES);
        return nfa->n_states == 0 ? RPQ_EINVAL : RPQ_EUNSUPPORTED;
    }
    if (nfa->n_labels == 0 || nfa->n_labels > g->L) {
        rpq::set_error("automaton has %u labels; the graph has %u", nfa->n_labels, g->L);
        return RPQ_EINVAL;
    }
    const uint32_t smask = nfa->n_states == 32 ? 0xFFFFFFFFu : ((1u << nfa->n_states) - 1);
    if ((nfa->initial_mask & ~smask) || (nfa->final_mask & ~smask)) {
        rpq::set_error("initial/final mask names states >= n_states");
        return RPQ_EINVAL;
    }
    for (uint32_t q = 0; q < RPQ_MAX_STATES; ++q)
        for (uint32_t l = 0; l < RPQ_MAX_LABELS; ++l) {
            const uint32_t d = nfa->delta[q * RPQ_MAX_LABELS + l];
            if (!d) continue;
            if (q >= nfa->n_states || l >= nfa->n_labels || (d & ~smask)) {
                rpq::set_error("delta[%u][%u] is outside the automaton", q, l);
                return RPQ_EINVAL;
            }
        }
    return RPQ_OK;
}

void to_dev_nfa(const rpq_nfa* nfa, uint32_t L, DevNfa* d) {
    std::memset(d, 0, sizeof *d);
    d->Q = nfa->n_states;
    d->L = L;
    d->init = nfa->initial_mask;
    d->final = nfa->final_mask;
    for (uint32_t q = 0; q < nfa->n_states; ++q)
        for (uint32_t l = 0; l < L; ++l) {
            const uint32_t m = l < nfa->n_labels ? nfa->delta[q * RPQ_MAX_LABELS + l] : 0;
            d->delta[q * L + l] = m;
            if (m) d->qlab[q] |= 1ull << l;
        }
}

// Default shape: about 64K sources with a bit in flight, in units of up to 2048 sources below 2^22
// vertices and 4096 from there (five queries a step, at 1024, 2048 and 4096: R-MAT 18, all pairs, 174, 152
// and 148 ms; R-MAT 23, 65,536 sources, 749, 647 and 628), entries of more than 16 items cut into slices
// (at 16, 32, 64 and 256: 152, 156, 159 and 164 ms; 628, 656, 656 and 697; raised on graphs where the slice
// buffers would outgrow a quarter of the bitmaps).  Units in flight are sized for 64 GB of the 288 GB
// device, and a unit of the default width may take up to 96 GB alone.
constexpr uint64_t kTargetInFlight = 65536;
constexpr uint64_t kWorkspaceBudget = 64ull << 30;
constexpr uint64_t kUnitBudget = 96ull << 30;
constexpr uint32_t kDefaultChunk = 16;
// Bitmaps of all vertices below this size are not worth the classes' launches: they are cleared in the
// same 10 us.
constexpr uint64_t kCompactBytes = 64ull << 20;
// Sources up to one word of bits run in one unit either way; up to eight words their order is not worth
// its launches.
constexpr uint64_t kCompactSources = 64;
constexpr uint64_t kOrderSources = 512;
constexpr uint64_t kFillRows = 1ull << 18;

uint32_t max_default_width(uint32_t V) { return V >= (1u << 22) ? 4096 : 2048; }

uint64_t unit_bytes(uint64_t rows, uint32_t W) {
    // Vis + Next + two frontier lists of rows + row ids
    return rows * (W / 8) * 4 + rows * 8;
}

uint32_t add_class(Plan* p, uint64_t labels, bool src, uint64_t bound) {
    for (uint32_t c = 0; c < p->n_classes; ++c)
        if (p->labels[c] == labels && (((p->src >> c) & 1) != 0) == src) return c;
    const uint32_t c = p->n_classes++;
    p->labels[c] = labels;
    p->bound[c] = bound;
    p->list_at[c] = p->verts;
    p->verts += bound;
    if (src) p->src |= 1ull << c;
    return c;
}

void make_plan(const rpq_graph* g, const rpq::Csr& csr, const rpq_nfa* nfa, uint64_t n_sources, bool keys, Plan* p) {
    std::memset(p, 0, sizeof *p);
    to_dev_nfa(nfa, g->L, &p->dn);
    DevNfa& d = p->dn;
    p->csr = &csr;
    p->n_words = ((uint64_t)g->V + 63) / 64;
    p->eps = (d.init & d.final) != 0;
    // A source without a bit may have its zero-length walk as a key, which only extraction could put in
    // its place among the others' keys: with keys and the empty word every source gets a bit.
    p->compact_src = n_sources > kCompactSources && !(keys && p->eps);
    for (uint32_t q = 0; q < d.Q; ++q)
        if ((d.init >> q) & 1) p->init_labels |= d.qlab[q];
    uint64_t entering[RPQ_MAX_STATES] = {};
    for (uint32_t q = 0; q < d.Q; ++q) {
        uint32_t max_succ = 0;
        for (uint32_t l = 0; l < g->L; ++l) {
            const uint32_t to = d.delta[q * g->L + l];
            max_succ = std::max(max_succ, (uint32_t)__builtin_popcount(to));
            for (uint32_t t = to; t; t &= t - 1) entering[__builtin_ctz(t)] |= 1ull << l;
        }
        p->desc_items += (uint64_t)max_succ * g->E;   // the in-CSR holds the same distinct edges
    }
    const uint64_t in_flight = std::min<uint64_t>(kTargetInFlight, (n_sources + 63) / 64 * 64);
    const bool compact = (uint64_t)d.Q * g->V * (in_flight / 8) * 2 > kCompactBytes;
    auto bound_of = [&](uint64_t labels, bool src) {
        uint64_t n = src ? n_sources : 0;
        for (uint64_t m = labels; m; m &= m - 1) n += csr.n_entered[__builtin_ctzll(m)];
        return std::min<uint64_t>(n, g->V);
    };
    auto worth = [&](uint64_t bound) { return bound <= (uint64_t)g->V * 3 / 4; };
    bool ans_all = !compact, ans_src = false;
    uint64_t ans_labels = 0;
    for (uint32_t q = 0; q < d.Q; ++q) {
        const bool init = (d.init >> q) & 1, fin = (d.final >> q) & 1;
        const uint64_t bound = bound_of(entering[q], init);
        d.kind[q] = ROW_ALL;
        p->rows[q] = g->V;
        if (!entering[q] && !init) {
            p->rows[q] = 0;   // nothing leads here
            continue;
        }
        if (compact && !entering[q]) {
            d.kind[q] = ROW_SOURCE;
            p->rows[q] = 0;
        } else if (compact && worth(bound)) {
            const uint32_t c = add_class(p, entering[q], init, bound);
            d.kind[q] = ROW_RANKED;
            d.rank_at[q] = (uint32_t)(c * p->n_words);
            d.list_at[q] = p->list_at[c];
            p->rows[q] = bound;
        }
        if (fin) {
            ans_labels |= entering[q];
            ans_src |= init;
            ans_all |= d.kind[q] == ROW_ALL;
        }
    }
    d.src_rank_at = kNone;
    for (uint32_t q = 0; q < d.Q; ++q)
        if (((d.final >> q) & 1) && d.kind[q] == ROW_SOURCE)
            d.src_rank_at = (uint32_t)(add_class(p, 0, true, std::min<uint64_t>(n_sources, g->V)) * p->n_words);
    d.ans_class = d.ans_rank_at = kNone;
    p->ans_bound = g->V;
    if (!ans_all && worth(bound_of(ans_labels, ans_src))) {
        p->ans_bound = bound_of(ans_labels, ans_src);
        d.ans_class = add_class(p, ans_labels, ans_src, p->ans_bound);
        d.ans_rank_at = (uint32_t)(d.ans_class * p->n_words);
        d.ans_list_at = p->list_at[d.ans_class];
    }
}

// Slot rows at unit width W, and where each state's begin.
uint64_t place_rows(const Plan& p, uint32_t W, uint32_t* base) {
    uint64_t r = 0;
    for (uint32_t q = 0; q < p.dn.Q; ++q) {
        if (base) base[q] = (uint32_t)r;
        r += p.dn.kind[q] == ROW_SOURCE ? W : p.rows[q];
    }
    if (base) base[p.dn.Q] = (uint32_t)r;
    return r;
}

// Width of a unit for n_bits sources.  Wide rows turn one visit of an edge into work for more sources, so
// one unit takes them all where it can: a second unit visits every edge again (R-MAT 22, about 300 sources
// with a bit: 11.5 ms at 64, 5.4 at 256, 4.0 at 512), and words that no source uses are still read and
// written (6.7 at 2048).  From 512 on, up to a quarter of a unit's sources rather go to a second unit.  A
// row has at least two words: at one, ORs to neighbouring rows from different dies meet in one line more
// often (R-MAT 18, about 30 sources: 0.57 ms at 64 and 0.56 at 128, 0.64 at 512).  On up to 2^13 vertices
// wide units are few rows, and a level of few rows does not fill the device: units widen there only while
// they have more than kFillRows rows together (by levels, all pairs of 2,000 vertices over a*: 0.67 ms at
// 128, 2.06 at 2048; of 8,192 vertices over (a|b)*.a.b: 9.4 ms at 128, 3.9 at 2048).
uint32_t default_width(const Plan& p, uint64_t n_bits, uint32_t V) {
    uint32_t W = 128;
    while (W < max_default_width(V) && (W < 512 ? W < n_bits : (uint64_t)W * 4 < n_bits * 3) &&
           (V > (1u << 13) || (n_bits + W - 1) / W * place_rows(p, W, nullptr) > kFillRows))
        W *= 2;
    while (W > 64 && unit_bytes(place_rows(p, W, nullptr), W) > kUnitBudget) W /= 2;
    return W;
}

// The part of k_small_search's conditions that the number of sources has no say in: its rows fit in LDS, every
// state has all its rows, and one block can visit all edges of a level.  A caller that sets a knob of the
// level kernels gets them.
bool small_graph(const Plan& p, const rpq_eval_opts* o) {
    if (o && (o->batch_width || o->concurrency || o->chunk_edges || o->sync_every || o->visit)) return false;
    if (place_rows(p, 64, nullptr) > kSmallRows || p.desc_items > kSmallItems) return false;
    for (uint32_t q = 0; q < p.dn.Q; ++q)
        if (p.dn.kind[q] != ROW_ALL) return false;
    return true;
}

// n_sources: the caller's; n_bits: those that get a bit (at most n_sources), which decides the shape.
int make_layout(const rpq_graph* g, const Plan& p, uint64_t n_sources, uint64_t n_bits, uint32_t flags,
                const rpq_eval_opts* o, bool noalloc, Layout* Lo) {
    Layout x;
    std::memset(&x, 0, sizeof x);
    x.Q = p.dn.Q;
    x.L = g->L;
    x.V = g->V;
    // the search in LDS takes 32 sources a block whatever the width, and its answers are read in narrow rows
    x.W = (o && o->batch_width) ? o->batch_width : small_graph(p, o) ? 128 : default_width(p, n_bits, g->V);
    if (x.W != 64 && x.W != 128 && x.W != 256 && x.W != 512 && x.W != 1024 && x.W != 2048 && x.W != 4096) {
        rpq::set_error("batch_width must be 64, 128, 256, 512, 1024, 2048 or 4096");
        return RPQ_EINVAL;
    }
    x.K = x.W / 64;
    x.H = (o && o->chunk_edges) ? o->chunk_edges : kDefaultChunk;
    // seen OR unless asked otherwise: the faster scheme on both R-MAT 18 and R-MAT 23 (the
    // expansion's comment has the figures)
    x.seen_or = (o && o->visit) ? o->visit == RPQ_VISIT_SEEN_OR : 1u;
    if (x.H > 65535) {
        rpq::set_error("chunk_edges must be <= 65535");
        return RPQ_EINVAL;
    }
    const bool auto_chunk = !(o && o->chunk_edges);
    x.sync_every = (o && o->sync_every) ? o->sync_every : 4;
    x.max_len = (flags & RPQ_LENGTH_BOUND) ? (uint64_t)o->max_length : ~0ull;
    const uint64_t units = std::max<uint64_t>(1, (n_bits + x.W - 1) / x.W);
    const uint64_t R = std::max<uint64_t>(1, place_rows(p, x.W, nullptr));
    const uint64_t bitmap_bytes = R * x.K * 8;
    // slices of one level and unit: entries with work > H take ceil(work / H) <= 2 work / H
    // each, and the work of all entries of state q is at most E * max |delta(q, l)|.
    // Default slice size: the smallest (fastest) that keeps a unit's two slice buffers within a
    // quarter of its bitmaps
    while (auto_chunk && x.H < 256 && 2 * (2 * p.desc_items / x.H + 2) * sizeof(Desc) > unit_bytes(R, x.W) / 4)
        x.H *= 2;
    const uint64_t desc_per_unit = 2 * p.desc_items / x.H + 2;
    uint64_t G = (o && o->concurrency) ? o->concurrency : 0;
    if (!G) {
        G = std::max<uint64_t>(1, kTargetInFlight / x.W);
        const uint64_t per_unit = unit_bytes(R, x.W) + 2 * desc_per_unit * sizeof(Desc);
        G = std::min<uint64_t>(G, std::max<uint64_t>(1, kWorkspaceBudget / per_unit));
    }
    G = std::min<uint64_t>(G, units);
    x.G = (uint32_t)G;
    x.list_cap = G * R;
    if (x.list_cap >= 0xFFFFFFFFull) {
        rpq::set_error("concurrency * states * vertices must stay below 2^32; lower concurrency");
        return RPQ_EUNSUPPORTED;
    }
    x.R = (uint32_t)R;
    x.desc_cap = G * desc_per_unit;
    // answer vertices per extraction wave: 4096, fewer while that leaves the device idle, and down to one
    // step of a wave on the smallest graphs (1,000 vertices, all pairs: tallies 40 us and keys 65 us at 256)
    const uint64_t ans = std::max<uint64_t>(1, p.ans_bound);
    x.chunk = 4096;
    while (x.chunk > 256 && G * ((x.K + 3) / 4) * ((ans + x.chunk - 1) / x.chunk) < 8192) x.chunk /= 2;
    while (x.chunk > 64 && G * ((x.K + 3) / 4) * ((ans + x.chunk - 1) / x.chunk) < 1024) x.chunk /= 2;
    x.nchunks = (uint32_t)((ans + x.chunk - 1) / x.chunk);
    uint64_t off = 0;
    auto take = [&](uint64_t bytes) {
        const uint64_t o2 = off;
        off = align256(off + bytes);
        return o2;
    };
    x.off_counters = take(C_NCOUNTERS * 8);
    x.off_tally = take((uint64_t)kMaxLevelBlocks * kTallyStride * 8);
    x.off_xtally = take((uint64_t)kMaxExtractBlocks * 2 * 8);
    x.off_src_bits = take(p.src ? p.n_words * 8 : 0);
    x.zero_words = off / 8;   // everything up to here starts at zero
    x.off_nfa = take(sizeof(DevNfa));
    x.off_tile_n = take((n_sources + kSrcTile - 1) / kSrcTile * 4);
    x.off_srcs = take(p.compact_src ? n_sources * 4 : 0);
    x.off_pos = take(p.compact_src ? n_sources * 4 : 0);
    // the ordered copies, and what ordering a group takes
    x.order = p.compact_src && n_sources > kOrderSources && !noalloc;
    const uint64_t n_order = x.order ? n_sources : 0;
    x.off_srcs2 = take(n_order * 4);
    x.off_pos2 = take(n_order * 4);
    x.off_bit_of = take(n_order * 4);
    x.off_hist = take(x.order ? (kScores + rpq::scan_temp_elems(kScores)) * 8 : 0);
    x.off_score = take(n_order * 8);
    x.off_rank = take(p.n_classes * p.n_words * 16);
    x.off_verts = take(p.verts * 4);
    x.off_class_n = take(p.n_classes * 4);
    x.off_class_tile_n = take(p.n_classes * ((p.n_words + 63) / 64) * 4);
    // With more than one group the visited bitmap is double-buffered: a group's answers are extracted
    // from it on a second stream while the next group's levels fill the other one.
    x.off_vis = take(G * bitmap_bytes);
    x.off_next = take(G * bitmap_bytes);
    x.off_vis2 = units > G && !noalloc ? take(G * bitmap_bytes) : x.off_vis;
    x.off_touch = take((G * R + 63) / 64 * 8);
    x.off_ever = take(x.seen_or ? (G * R + 63) / 64 * 8 : 0);
    x.off_fresh = take(x.seen_or ? (G * R + 63) / 64 * 8 : 0);
    x.off_full = take((G * R + 7) / 8 * 8);
    x.off_active = take(2 * G * x.K * 8);
    for (int i = 0; i < 2; ++i) {
        x.off_ids[i] = take(x.list_cap * 4);
        x.off_rows[i] = take(x.list_cap * x.K * 8);
        x.off_desc[i] = take(x.desc_cap * sizeof(Desc));
    }
    x.off_acc = take(G * x.W * 16);
    const bool want_pairs = (flags & RPQ_PAIRS) != 0;
    x.off_partial = take(want_pairs ? G * x.W * (uint64_t)x.nchunks * 4 : 0);
    x.off_srcbase = take(want_pairs ? G * x.W * 8 : 0);
    x.total = off;
    *Lo = x;
    return RPQ_OK;
}

Args make_args(const rpq_graph* g, const Plan& p, const Layout& x, char* ws) {
    Args a;
    std::memset(&a, 0, sizeof a);
    a.row_ptr = p.csr->row_ptr;
    a.dst = p.csr->dst;
    a.lmask = p.csr->lmask;
    a.nfa = reinterpret_cast<const DevNfa*>(ws + x.off_nfa);
    a.rank = reinterpret_cast<const ulonglong2*>(ws + x.off_rank);
    a.verts = reinterpret_cast<const uint32_t*>(ws + x.off_verts);
    a.class_n = reinterpret_cast<const uint32_t*>(ws + x.off_class_n);
    a.vis = reinterpret_cast<uint64_t*>(ws + x.off_vis);
    a.next = reinterpret_cast<uint64_t*>(ws + x.off_next);
    a.touch = reinterpret_cast<uint64_t*>(ws + x.off_touch);
    a.ever = reinterpret_cast<uint64_t*>(ws + x.off_ever);
    a.fresh = reinterpret_cast<uint64_t*>(ws + x.off_fresh);
    a.full = reinterpret_cast<uint8_t*>(ws + x.off_full);
    a.active = reinterpret_cast<uint64_t*>(ws + x.off_active);
    a.n_active = (uint64_t)x.G * x.K;
    a.ids0 = reinterpret_cast<uint32_t*>(ws + x.off_ids[0]);
    a.ids1 = reinterpret_cast<uint32_t*>(ws + x.off_ids[1]);
    a.rows0 = reinterpret_cast<uint64_t*>(ws + x.off_rows[0]);
    a.rows1 = reinterpret_cast<uint64_t*>(ws + x.off_rows[1]);
    a.desc0 = reinterpret_cast<Desc*>(ws + x.off_desc[0]);
    a.desc1 = reinterpret_cast<Desc*>(ws + x.off_desc[1]);
    a.counters = reinterpret_cast<unsigned long long*>(ws + x.off_counters);
    a.tally = reinterpret_cast<unsigned long long*>(ws + x.off_tally);
    a.xtally = reinterpret_cast<unsigned long long*>(ws + x.off_xtally);
    a.V = x.V;
    a.L = x.L;
    a.Q = x.Q;
    a.H = x.H;
    a.R = x.R;
    a.W = x.W;
    a.seen_or = x.seen_or;
    a.list_cap = x.list_cap;
    a.desc_cap = x.desc_cap;
    return a;
}

// Grid of a level kernel: as many blocks as the device keeps resident at once (the kernels
// stride over their work, so a grid beyond residency would only add a tail round).
unsigned resident_grid(const void* kernel) {
    int dev = 0, n_cu = 0, per_cu = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, kBlock, 0) != hipSuccess || n_cu <= 0 ||
        per_cu <= 0)
        return 2048;
    return std::min((unsigned)(n_cu * per_cu), kMaxLevelBlocks);
}

template <int K>
struct LevelGrids {
    unsigned expand, expand_seen, compact, finalize, finalize_seen;
    static const LevelGrids& get() {
        static const LevelGrids g{resident_grid(reinterpret_cast<const void*>(&k_expand<K, false>)),
                                  resident_grid(reinterpret_cast<const void*>(&k_expand<K, true>)),
                                  resident_grid(reinterpret_cast<const void*>(&k_compact)),
                                  resident_grid(reinterpret_cast<const void*>(&k_finalize<K, false>)),
                                  resident_grid(reinterpret_cast<const void*>(&k_finalize<K, true>))};
        return g;
    }
};

// Process-wide profiling state: event pairs around level kernels, resolved at
// the host synchronisation points of rpq_eval.
struct Profiler {
    std::mutex mu;
    bool on = false;
    rpq_profile acc{};
    std::vector<hipEvent_t> pool;
    std::vector<std::pair<hipEvent_t, hipEvent_t>> pend_expand, pend_finalize, pend_extract;

    hipEvent_t get() {
        if (!pool.empty()) {
            hipEvent_t e = pool.back();
            pool.pop_back();
            return e;
        }
        hipEvent_t e = nullptr;
        if (hipEventCreate(&e) != hipSuccess) return nullptr;
        return e;
    }
    // caller holds mu and has synchronised the stream(s) the events were recorded on; extraction
    // events (second stream) only when with_extract
    void resolve(bool with_extract = false) {
        if (with_extract) {
            for (auto& pr : pend_extract) {
                float ms = 0.f;
                if (hipEventElapsedTime(&ms, pr.first, pr.second) == hipSuccess) {
                    acc.extract_ms += ms;
                    acc.extract_launches++;
                }
                pool.push_back(pr.first);
                pool.push_back(pr.second);
            }
            pend_extract.clear();
        }
        for (int which = 0; which < 2; ++which) {
            auto& v = which ? pend_finalize : pend_expand;
            for (auto& pr : v) {
                float ms = 0.f;
                if (hipEventElapsedTime(&ms, pr.first, pr.second) == hipSuccess) {
                    if (which) {
                        acc.finalize_ms += ms;
                        acc.finalize_launches++;
                    } else {
                        acc.expand_ms += ms;
                        acc.expand_launches++;
                    }
                }
                // the expansion's end event is also the finalize's start event:
                // return each event to the pool exactly once
                if (which) {
                    pool.push_back(pr.first);
                    pool.push_back(pr.second);
                } else {
                    pool.push_back(pr.first);
                }
            }
            v.clear();
        }
    }
};

Profiler& profiler() {
    static Profiler* p = new Profiler();
    return *p;
}

// a wave takes 64 words of 64 rows
template <int K>
unsigned compact_grid(uint64_t n_rows) {
    const uint64_t per_block = 4096 * kWaves;
    return (unsigned)std::min<uint64_t>(LevelGrids<K>::get().compact, (n_rows + per_block - 1) / per_block);
}

template <int K>
int launch_level(const Args& a, int p, uint64_t n_rows, uint32_t level, int count_work, bool may_profile,
                 hipStream_t s) {
    Profiler& pr = profiler();
    const bool on = may_profile && pr.on;
    hipEvent_t e0 = nullptr, e1 = nullptr, e2 = nullptr;
    if (on) {
        std::lock_guard<std::mutex> lk(pr.mu);
        e0 = pr.get();
        e1 = pr.get();
        e2 = pr.get();
    }
    if (e0) RPQ_HIP(hipEventRecord(e0, s));
    if (a.seen_or)
        hipLaunchKernelGGL((k_expand<K, true>), dim3(LevelGrids<K>::get().expand_seen), dim3(kBlock), 0, s, a, p);
    else
        hipLaunchKernelGGL((k_expand<K, false>), dim3(LevelGrids<K>::get().expand), dim3(kBlock), 0, s, a, p);
    RPQ_LAUNCH_CHECK();
    if (e1) RPQ_HIP(hipEventRecord(e1, s));
    hipLaunchKernelGGL(k_compact, dim3(compact_grid<K>(n_rows)), dim3(kBlock), 0, s, a, p, n_rows, level);
    RPQ_LAUNCH_CHECK();
    if (a.seen_or)
        hipLaunchKernelGGL((k_finalize<K, true>), dim3(LevelGrids<K>::get().finalize_seen), dim3(kBlock), 0, s, a, p,
                           count_work);
    else
        hipLaunchKernelGGL((k_finalize<K, false>), dim3(LevelGrids<K>::get().finalize), dim3(kBlock), 0, s, a, p,
                           count_work);
    RPQ_LAUNCH_CHECK();
    if (e2) RPQ_HIP(hipEventRecord(e2, s));
    if (on && e0 && e1 && e2) {
        std::lock_guard<std::mutex> lk(pr.mu);
        pr.pend_expand.emplace_back(e0, e1);
        pr.pend_finalize.emplace_back(e1, e2);
    }
    return RPQ_OK;
}

void profile_resolve() {
    Profiler& pr = profiler();
    std::lock_guard<std::mutex> lk(pr.mu);
    pr.resolve();
}

template <int K>
int launch_finalize(const Args& a, int p, uint64_t n_rows, uint32_t level, int count_work, hipStream_t s) {
    hipLaunchKernelGGL(k_compact, dim3(compact_grid<K>(n_rows)), dim3(kBlock), 0, s, a, p, n_rows, level);
    RPQ_LAUNCH_CHECK();
    if (a.seen_or)
        hipLaunchKernelGGL((k_finalize<K, true>), dim3(LevelGrids<K>::get().finalize_seen), dim3(kBlock), 0, s, a, p,
                           count_work);
    else
        hipLaunchKernelGGL((k_finalize<K, false>), dim3(LevelGrids<K>::get().finalize), dim3(kBlock), 0, s, a, p,
                           count_work);
    RPQ_LAUNCH_CHECK();
    return RPQ_OK;
}

// A second stream for extraction (one per host thread and device, created on first use and kept
// for the thread's lifetime) and the events that order its work against the caller's stream.  The
// destructor drains the side stream, so no work of a call outlives it on any return path.  Without
// a side stream (creation failed) everything runs on the caller's stream, in the same order.
struct SideStream {
    static constexpr int kMaxDevices = 64;
    hipStream_t stream = nullptr;
    hipEvent_t leveled = nullptr;
    hipEvent_t extracted[2] = {nullptr, nullptr};

    explicit SideStream(bool want) {
        if (!want) return;
        static thread_local hipStream_t per_device[kMaxDevices] = {};
        int dev = 0;
        if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return;
        if (!per_device[dev] && hipStreamCreateWithFlags(&per_device[dev], hipStreamNonBlocking) != hipSuccess) {
            per_device[dev] = nullptr;
            return;
        }
        if (hipEventCreateWithFlags(&leveled, hipEventDisableTiming) != hipSuccess ||
            hipEventCreateWithFlags(&extracted[0], hipEventDisableTiming) != hipSuccess ||
            hipEventCreateWithFlags(&extracted[1], hipEventDisableTiming) != hipSuccess) {
            destroy_events();
            return;
        }
        stream = per_device[dev];
    }
    ~SideStream() {
        if (stream) (void)hipStreamSynchronize(stream);
        destroy_events();
    }
    void destroy_events() {
        if (leveled) (void)hipEventDestroy(leveled);
        for (hipEvent_t& e : extracted)
            if (e) (void)hipEventDestroy(e);
        leveled = nullptr;
        extracted[0] = extracted[1] = nullptr;
    }
    SideStream(const SideStream&) = delete;
    SideStream& operator=(const SideStream&) = delete;
};

template <int K>
int launch_extract(const Args& a, int mode, const ExtractArgs& e, hipStream_t s) {
    const uint64_t waves = (uint64_t)e.G * (K / kExtractWords<K>()) * e.nchunks;
    const uint64_t blocks = (waves + kWaves - 1) / kWaves;
    const dim3 grid((unsigned)std::min<uint64_t>(blocks, mode == X_TOTALS ? kMaxExtractBlocks : 16384));
    if (mode == X_KEYS) hipLaunchKernelGGL((k_extract<K, X_KEYS>), grid, dim3(kBlock), 0, s, a, e);
    else if (mode == X_TALLIES) hipLaunchKernelGGL((k_extract<K, X_TALLIES>), grid, dim3(kBlock), 0, s, a, e);
    else hipLaunchKernelGGL((k_extract<K, X_TOTALS>), grid, dim3(kBlock), 0, s, a, e);
    RPQ_LAUNCH_CHECK();
    return RPQ_OK;
}

#define RPQ_DISPATCH_K(K, CALL)                                      \
    switch (K) {                                                     \
        case 1: { constexpr int KK = 1; CALL; } break;               \
        case 2: { constexpr int KK = 2; CALL; } break;               \
        case 4: { constexpr int KK = 4; CALL; } break;               \
        case 8: { constexpr int KK = 8; CALL; } break;               \
        case 16: { constexpr int KK = 16; CALL; } break;             \
        case 32: { constexpr int KK = 32; CALL; } break;             \
        case 64: { constexpr int KK = 64; CALL; } break;             \
        default: rpq::set_error("bad batch width"); return RPQ_EINVAL; \
    }

// A copy stream per host thread and device (created on first use, kept for the thread's lifetime).
hipStream_t copy_stream() {
    constexpr int kMaxDevices = 64;
    static thread_local hipStream_t per_device[kMaxDevices] = {};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return nullptr;
    if (!per_device[dev] && hipStreamCreateWithFlags(&per_device[dev], hipStreamNonBlocking) != hipSuccess)
        per_device[dev] = nullptr;
    return per_device[dev];
}

// Host side of rpq_eval_stream.  A counted group's keys [next_key, end_key) are cut into windows of
// at most chunk_keys keys; window i is extracted into device chunk i % 2 on the extraction stream,
// copied to host chunk i % 2 on the copy stream, and handed to the sink once its copy is complete.
// At most two windows are in flight, so a chunk is rewritten only after the sink has returned for
// the window it held.  Windows are issued in key order and delivered in issue order.
struct PairStreamer {
    const rpq_pair_stream* ps = nullptr;
    hipStream_t xs = nullptr, cs = nullptr;
    hipEvent_t ext_done[2] = {nullptr, nullptr}, copied[2] = {nullptr, nullptr}, counted = nullptr;
    uint64_t* gend = nullptr;   // pinned: key index at which the counted group ends
    // the group whose windows are being issued
    bool pending = false, end_known = false;
    uint64_t next_key = 0, end_key = 0;
    hipEvent_t group_done = nullptr;   // recorded on xs after the group's last window
    Args ga;
    ExtractArgs ge;
    uint32_t K = 0;
    // windows issued and not yet delivered: a ring of two, oldest at head
    int win_buf[2] = {0, 0};
    uint64_t win_n[2] = {0, 0};
    int head = 0, n_inflight = 0, next_buf = 0;
    uint64_t delivered = 0;
    uint64_t* written = nullptr;   // the caller's result->written, kept current

    PairStreamer() = default;
    PairStreamer(const PairStreamer&) = delete;
    PairStreamer& operator=(const PairStreamer&) = delete;

    int init(const rpq_pair_stream* p, hipStream_t extraction, uint64_t* pinned_slot, uint64_t* written_out) {
        ps = p;
        written = written_out;
        xs = extraction;
        cs = copy_stream();
        if (!cs) cs = xs;
        gend = pinned_slot;
        for (int b = 0; b < 2; ++b) {
            RPQ_HIP(hipEventCreateWithFlags(&ext_done[b], hipEventDisableTiming));
            RPQ_HIP(hipEventCreateWithFlags(&copied[b], hipEventDisableTiming));
        }
        RPQ_HIP(hipEventCreateWithFlags(&counted, hipEventDisableTiming));
        return RPQ_OK;
    }
    ~PairStreamer() {
        // no work of the call outlives it, whatever the return path
        if (cs) (void)hipStreamSynchronize(cs);
        if (xs) (void)hipStreamSynchronize(xs);
        for (hipEvent_t e : {ext_done[0], ext_done[1], copied[0], copied[1], counted})
            if (e) (void)hipEventDestroy(e);
    }

    // The keys of a group whose count pass and per-source offsets are enqueued on xs; `done` is
    // recorded on xs once its last window is issued.
    int start_group(const Args& a, const ExtractArgs& e, uint32_t K_, hipEvent_t done) {
        RPQ_HIP(hipMemcpyAsync(gend, a.counters + C_PAIRBASE, 8, hipMemcpyDeviceToHost, xs));
        RPQ_HIP(hipEventRecord(counted, xs));
        pending = true;
        end_known = false;
        next_key = end_key;   // this group's keys follow the previous group's
        group_done = done;
        ga = a;
        ge = e;
        K = K_;
        return RPQ_OK;
    }

    int deliver_head() {
        const int b = win_buf[head];
        const uint64_t n = win_n[head];
        head ^= 1;
        --n_inflight;
        if (ps->sink(ps->host_chunks + (uint64_t)b * ps->chunk_keys, n, ps->user) != 0) {
            rpq::set_error("the pair sink stopped the evaluation after %llu keys", (unsigned long long)delivered);
            return RPQ_ECANCELED;
        }
        delivered += n;
        if (written) *written = delivered;
        return RPQ_OK;
    }

    // hand every completed window to the sink; with wait, block for the oldest one first
    int deliver(bool wait) {
        while (n_inflight) {
            const hipEvent_t e = copied[win_buf[head]];
            if (wait) {
                RPQ_HIP(hipEventSynchronize(e));
                wait = false;
            } else {
                const hipError_t q = hipEventQuery(e);
                if (q == hipErrorNotReady) break;
                if (q != hipSuccess) {
                    rpq::set_error("HIP error in hipEventQuery: %s", hipGetErrorString(q));
                    return RPQ_EDEVICE;
                }
            }
            RPQ_TRY(deliver_head());
        }
        return RPQ_OK;
    }

    int issue_window() {
        const int b = next_buf;
        next_buf ^= 1;
        const uint64_t n = std::min<uint64_t>(ps->chunk_keys, end_key - next_key);
        uint64_t* dev = ps->device_chunks + (uint64_t)b * ps->chunk_keys;
        ge.pairs = dev;
        ge.off = next_key;
        ge.cap = n;
        RPQ_DISPATCH_K(K, RPQ_TRY(launch_extract<KK>(ga, X_KEYS, ge, xs)));
        RPQ_HIP(hipEventRecord(ext_done[b], xs));
        RPQ_HIP(hipStreamWaitEvent(cs, ext_done[b], 0));
        RPQ_HIP(hipMemcpyAsync(ps->host_chunks + (uint64_t)b * ps->chunk_keys, dev, n * 8, hipMemcpyDeviceToHost, cs));
        RPQ_HIP(hipEventRecord(copied[b], cs));
        const int slot = (head + n_inflight) & 1;
        win_buf[slot] = b;
        win_n[slot] = n;
        ++n_inflight;
        next_key += n;
        return RPQ_OK;
    }

    // Deliver what is complete and issue what fits.  With finish, return only once every window of
    // the pending group is issued: its visited bitmap and per-source arrays may then be reused by work
    // enqueued on xs after this point (or ordered after group_done).
    int pump(bool finish) {
        for (;;) {
            RPQ_TRY(deliver(false));
            if (!pending) return RPQ_OK;
            if (!end_known) {
                if (finish) {
                    RPQ_HIP(hipEventSynchronize(counted));
                } else {
                    const hipError_t q = hipEventQuery(counted);
                    if (q == hipErrorNotReady) return RPQ_OK;
                    if (q != hipSuccess) {
                        rpq::set_error("HIP error in hipEventQuery: %s", hipGetErrorString(q));
                        return RPQ_EDEVICE;
                    }
                }
                end_key = *gend;
                end_known = true;
            }
            while (n_inflight < 2 && next_key < end_key) RPQ_TRY(issue_window());
            if (next_key == end_key) {
                if (group_done) RPQ_HIP(hipEventRecord(group_done, xs));
                pending = false;
                return RPQ_OK;
            }
            if (!finish) return RPQ_OK;
            RPQ_TRY(deliver(true));
        }
    }

    // every window issued and delivered
    int drain() {
        RPQ_TRY(pump(true));
        while (n_inflight) RPQ_TRY(deliver(true));
        return RPQ_OK;
    }
};

int prepare(rpq_graph_t g, const rpq_nfa* nfa_in, uint64_t n_sources, uint32_t flags, const rpq_eval_opts* opts,
            Plan* plan, Layout* lay, bool noalloc = false) {
    if (!g) {
        rpq::set_error("graph is NULL");
        return RPQ_EINVAL;
    }
    if (flags & ~(RPQ_PAIRS | RPQ_PER_SOURCE | RPQ_ALL_SOURCES | RPQ_REVERSE | RPQ_SPARSE | RPQ_LENGTH_BOUND)) {
        rpq::set_error("unknown flags 0x%x", flags);
        return RPQ_EINVAL;
    }
    if ((flags & RPQ_LENGTH_BOUND) && !opts) {
        rpq::set_error("RPQ_LENGTH_BOUND needs opts->max_length");
        return RPQ_EINVAL;
    }
    if (opts && opts->visit > RPQ_VISIT_SEEN_OR) {
        rpq::set_error("rpq_eval_opts.visit must be 0, RPQ_VISIT_TWO_READS or RPQ_VISIT_SEEN_OR");
        return RPQ_EINVAL;
    }
    RPQ_TRY(validate_nfa(g, nfa_in));
    if ((flags & RPQ_REVERSE) && !g->has_in) {
        rpq::set_error("RPQ_REVERSE needs a graph built with RPQ_BUILD_IN_CSR");
        return RPQ_EUNSUPPORTED;
    }
    rpq_nfa rev;
    if (flags & RPQ_REVERSE) RPQ_TRY(rpq_nfa_reverse(nfa_in, &rev));
    make_plan(g, (flags & RPQ_REVERSE) ? g->in : g->out, (flags & RPQ_REVERSE) ? &rev : nfa_in, n_sources,
              (flags & RPQ_PAIRS) != 0, plan);
    return make_layout(g, *plan, n_sources, n_sources, flags, opts, noalloc, lay);
}

}  // namespace

extern "C" {

int rpq_eval_workspace_size(rpq_graph_t g, const rpq_nfa* nfa, uint64_t n_sources, uint32_t flags,
                            const rpq_eval_opts* opts, uint64_t* bytes) {
    rpq::clear_error();
    if (!bytes) {
        rpq::set_error("bytes is NULL");
        return RPQ_EINVAL;
    }
    if (g && (flags & RPQ_ALL_SOURCES) && n_sources == 0) n_sources = g->V;
    if (flags & RPQ_SPARSE) return rpq::sparse_workspace_size(g, nfa, n_sources, flags, bytes);
    Plan plan;
    Layout lay;
    RPQ_TRY(prepare(g, nfa, n_sources, flags, opts, &plan, &lay));
    *bytes = lay.total;
    return RPQ_OK;
}

int rpq_eval(rpq_graph_t g, const rpq_nfa* nfa, const uint32_t* sources, uint64_t n_sources, uint32_t flags,
             const rpq_eval_opts* opts, void* workspace, uint64_t workspace_bytes, rpq_result* res,
             hipStream_t stream) {
    rpq::clear_error();
    const int rc =
        rpq::eval_impl(g, nfa, sources, n_sources, flags, opts, nullptr, workspace, workspace_bytes, res, stream);
    // a failing call may leave kernels of its own queued on the stream: drain them, so that the
    // caller may reuse or release the workspace as soon as the call returns
    if (rc != RPQ_OK && rc != RPQ_EOVERFLOW) (void)hipStreamSynchronize(stream);
    return rc;
}

}  // extern "C"

namespace {

// Whether k_small_search takes the call.
bool small_search(const Plan& p, const Layout& x, uint64_t n_bits, const rpq_eval_opts* o) {
    return small_graph(p, o) && n_bits != 0 && n_bits <= (uint64_t)x.G * x.W &&
           (uint64_t)x.G * (x.W / 32) <= kMaxLevelBlocks;
}

// The plain evaluation.  With noalloc the call creates nothing: counters are read into a
// pageable stack buffer instead of the thread's pinned staging buffer, extraction stays on the
// caller's stream (the layout then holds a single visited bitmap), and no profiling events are
// recorded.
int eval_core(rpq_graph_t g, const rpq_nfa* nfa, const uint32_t* sources, uint64_t n_sources, uint32_t flags,
              const rpq_eval_opts* opts, const uint64_t* target, void* workspace, uint64_t workspace_bytes,
              rpq_result* res, hipStream_t stream, bool noalloc, const rpq_pair_stream* ps = nullptr) {
    if (!res) {
        rpq::set_error("result is NULL");
        return RPQ_EINVAL;
    }
    if (g && (flags & RPQ_ALL_SOURCES)) {
        if (sources) {
            rpq::set_error("RPQ_ALL_SOURCES requires sources == NULL");
            return RPQ_EINVAL;
        }
        if (n_sources == 0) n_sources = g->V;
        if (n_sources != g->V) {
            rpq::set_error("RPQ_ALL_SOURCES requires n_sources == n_vertices");
            return RPQ_EINVAL;
        }
    } else if (n_sources && !sources) {
        rpq::set_error("sources is NULL");
        return RPQ_EINVAL;
    }
    if (!ps && (flags & RPQ_PAIRS) && res->capacity && !res->pairs) {
        rpq::set_error("RPQ_PAIRS with a NULL pair buffer");
        return RPQ_EINVAL;
    }
    if ((flags & RPQ_PER_SOURCE) && n_sources && !res->per_source) {
        rpq::set_error("RPQ_PER_SOURCE with a NULL per_source buffer");
        return RPQ_EINVAL;
    }
    res->workspace_needed = 0;
    if ((flags & RPQ_LENGTH_BOUND) && !opts) {
        rpq::set_error("RPQ_LENGTH_BOUND needs opts->max_length");
        return RPQ_EINVAL;
    }
    if (flags & RPQ_SPARSE) {
        if (target) {
            rpq::set_error("internal: a result filter is not supported with RPQ_SPARSE");
            return RPQ_EINVAL;
        }
        if (flags & ~(RPQ_PAIRS | RPQ_PER_SOURCE | RPQ_ALL_SOURCES | RPQ_REVERSE | RPQ_SPARSE | RPQ_LENGTH_BOUND)) {
            rpq::set_error("unknown flags 0x%x", flags);
            return RPQ_EINVAL;
        }
        const uint64_t max_len = (flags & RPQ_LENGTH_BOUND) ? (uint64_t)opts->max_length : ~0ull;
        return rpq::sparse_eval(g, nfa, sources, n_sources, flags, max_len, workspace, workspace_bytes, res, stream);
    }
    Plan plan;
    Layout x;
    // streamed keys need the per-source offsets of the pairs layout
    if (ps) flags |= RPQ_PAIRS;
    RPQ_TRY(prepare(g, nfa, n_sources, flags, opts, &plan, &x, noalloc));
    if (!workspace || workspace_bytes < x.total) {
        rpq::set_error("workspace of %llu bytes is smaller than the %llu bytes needed",
                       (unsigned long long)workspace_bytes, (unsigned long long)x.total);
        res->workspace_needed = x.total;
        return RPQ_ENOMEM;
    }
    if (reinterpret_cast<uintptr_t>(workspace) & 255) {
        rpq::set_error("workspace must be 256-byte aligned");
        return RPQ_EINVAL;
    }
    const bool want_pairs = !ps && (flags & RPQ_PAIRS) && res->pairs != nullptr;
    res->written = res->count = res->hash = res->product_edges = res->levels = res->max_depth = 0;
    if (n_sources == 0) return RPQ_OK;

    char* ws = reinterpret_cast<char*>(workspace);
    Args a = make_args(g, plan, x, ws);
    uint64_t local_stage[C_NCOUNTERS];
    uint64_t* stage = noalloc ? local_stage : rpq::host_stage();
    if (!stage) {
        rpq::set_error("pinned host staging memory is unavailable");
        return RPQ_EDEVICE;
    }
    // 1. the sources (validity, which of them get a bit) and the classes
    RPQ_TRY(rpq::fill_u64(reinterpret_cast<uint64_t*>(ws), x.zero_words, 0, stream));
    SrcArgs sa;
    std::memset(&sa, 0, sizeof sa);
    sa.sources = sources;
    sa.n = n_sources;
    sa.lmask = plan.csr->lmask;
    sa.init_labels = plan.init_labels;
    sa.V = x.V;
    sa.compact = plan.compact_src ? 1 : 0;
    sa.eps = plan.eps ? 1 : 0;
    sa.target = target;
    sa.per_source = (flags & RPQ_PER_SOURCE) ? res->per_source : nullptr;
    sa.bits = plan.src ? reinterpret_cast<unsigned long long*>(ws + x.off_src_bits) : nullptr;
    sa.tile_n = reinterpret_cast<uint32_t*>(ws + x.off_tile_n);
    sa.out_srcs = reinterpret_cast<uint32_t*>(ws + x.off_srcs);
    sa.out_pos = reinterpret_cast<uint32_t*>(ws + x.off_pos);
    sa.counters = a.counters;
    const dim3 src_grid((unsigned)((n_sources + kSrcTile - 1) / kSrcTile));
    hipLaunchKernelGGL(k_src_count, src_grid, dim3(kBlock), 0, stream, sa);
    RPQ_LAUNCH_CHECK();
    if (plan.compact_src) {
        hipLaunchKernelGGL(k_src_write, src_grid, dim3(kBlock), 0, stream, sa);
        RPQ_LAUNCH_CHECK();
    }
    if (plan.n_classes) {
        ClassArgs ca;
        std::memset(&ca, 0, sizeof ca);
        std::memcpy(ca.labels, plan.labels, sizeof ca.labels);
        std::memcpy(ca.list_at, plan.list_at, sizeof ca.list_at);
        ca.src = plan.src;
        ca.entered = plan.csr->entered;
        ca.src_bits = sa.bits;
        ca.n_words = plan.n_words;
        ca.n_tiles = (uint32_t)((plan.n_words + 63) / 64);
        ca.tile_n = reinterpret_cast<uint32_t*>(ws + x.off_class_tile_n);
        ca.rank = reinterpret_cast<ulonglong2*>(ws + x.off_rank);
        ca.verts = reinterpret_cast<uint32_t*>(ws + x.off_verts);
        ca.class_n = reinterpret_cast<uint32_t*>(ws + x.off_class_n);
        const dim3 cgrid((ca.n_tiles + kWaves - 1) / kWaves, plan.n_classes);
        hipLaunchKernelGGL(k_class_count, cgrid, dim3(kBlock), 0, stream, ca);
        RPQ_LAUNCH_CHECK();
        hipLaunchKernelGGL(k_class_write, cgrid, dim3(kBlock), 0, stream, ca);
        RPQ_LAUNCH_CHECK();
    }
    RPQ_HIP(hipMemcpyAsync(stage, a.counters, C_NCOUNTERS * 8, hipMemcpyDeviceToHost, stream));
    RPQ_HIP(hipStreamSynchronize(stream));
    if (stage[C_ERR] & ERR_SOURCES) {
        rpq::set_error("sources must be strictly ascending vertex ids below n_vertices");
        return RPQ_EINVAL;
    }

    // 2. the shape for the sources that have a bit (the planned one where that needs more room)
    const uint64_t n_bits = plan.compact_src ? stage[C_ALIVE] : n_sources;
    if (n_bits < n_sources) {
        Layout y;
        RPQ_TRY(make_layout(g, plan, n_sources, n_bits, flags, opts, noalloc, &y));
        if (y.total <= workspace_bytes) x = y;
        a = make_args(g, plan, x, ws);
    }
    place_rows(plan, x.W, plan.dn.base);
    RPQ_HIP(hipMemcpyAsync(ws + x.off_nfa, &plan.dn, sizeof plan.dn, hipMemcpyHostToDevice, stream));
    a.target = target;
    const bool small = small_search(plan, x, n_bits, opts);
    const bool order = x.order && n_bits > kOrderSources && !small;
    OrderArgs oa;
    std::memset(&oa, 0, sizeof oa);
    oa.row_ptr = a.row_ptr;
    oa.dst = a.dst;
    oa.lmask = a.lmask;
    oa.init_labels = plan.init_labels;
    oa.L = x.L;
    oa.in_srcs = sa.out_srcs;
    oa.in_pos = sa.out_pos;
    oa.srcs = reinterpret_cast<uint32_t*>(ws + x.off_srcs2);
    oa.pos = reinterpret_cast<uint32_t*>(ws + x.off_pos2);
    oa.bit_of = reinterpret_cast<uint32_t*>(ws + x.off_bit_of);
    oa.hist = reinterpret_cast<uint64_t*>(ws + x.off_hist);
    oa.score = reinterpret_cast<uint32_t*>(ws + x.off_score);
    oa.rank = oa.score + n_sources;
    a.srcs = order ? oa.srcs : plan.compact_src ? sa.out_srcs : sources;
    a.pos = order ? oa.pos : plan.compact_src ? sa.out_pos : nullptr;
    a.bit_of = order ? oa.bit_of : nullptr;
    a.n_srcs = n_bits;
    const uint64_t bitmap_words = (uint64_t)x.R * x.K;   // of one unit
    if (!small) RPQ_TRY(rpq::fill_u64(a.touch, ((uint64_t)x.G * x.R + 63) / 64, 0, stream));
    if (!x.seen_or) RPQ_TRY(rpq::fill_u64(a.next, x.G * bitmap_words, 0, stream));

    const uint64_t per_group = (uint64_t)x.G * x.W;
    const uint64_t n_groups = (n_bits + per_group - 1) / per_group;
    const bool tallies = want_pairs || ps || (flags & RPQ_PER_SOURCE);
    ExtractArgs ea;
    std::memset(&ea, 0, sizeof ea);
    ea.nchunks = x.nchunks;
    ea.chunk = x.chunk;
    ea.acc = reinterpret_cast<unsigned long long*>(ws + x.off_acc);
    ea.partial = want_pairs || ps ? reinterpret_cast<uint32_t*>(ws + x.off_partial) : nullptr;
    uint64_t* srcbase = want_pairs || ps ? reinterpret_cast<uint64_t*>(ws + x.off_srcbase) : nullptr;
    ea.srcbase = srcbase;
    uint64_t final_rows = 0;
    for (uint32_t q = 0; q < x.Q; ++q)
        if ((plan.dn.final >> q) & 1) final_rows += plan.rows[q];
    // sources without a bit still have their zero-length level, if there is a state to start in
    uint64_t levels_total = n_bits || !plan.dn.init ? 0 : 1, max_depth = 0;
    // Extraction of group g runs on a second stream (xs) while the levels of group g + 1 run on
    // `stream` into the other visited bitmap: the level kernels are bound by memory, extraction by its
    // instruction stream.  Events order each bitmap's reuse and the final join.
    uint64_t* const vis_buf[2] = {reinterpret_cast<uint64_t*>(ws + x.off_vis),
                                  reinterpret_cast<uint64_t*>(ws + x.off_vis2)};
    const bool overlap = n_groups > 1 && x.off_vis2 != x.off_vis && !noalloc;
    SideStream side(overlap);
    hipStream_t xs = side.stream ? side.stream : stream;
    // streamed keys: windows of group g are extracted on xs while group g + 1's levels run; the
    // group-end key index is read through the pinned staging buffer, past the counter words
    PairStreamer st;
    if (ps) RPQ_TRY(st.init(ps, xs, stage + 64, &res->written));
    for (uint64_t grp = 0; grp < n_groups; ++grp) {
        const uint64_t gbase = grp * per_group;
        const uint64_t n_here = std::min<uint64_t>(per_group, n_bits - gbase);
        const uint32_t G_eff = (uint32_t)((n_here + x.W - 1) / x.W);
        const int buf = side.stream ? (int)(grp & 1) : 0;
        a.gbase = gbase;
        a.vis = vis_buf[buf];
        ea.G = G_eff;
        if (order) {
            oa.gbase = gbase;
            oa.n = n_here;
            const dim3 og((unsigned)((n_here + kBlock - 1) / kBlock));
            RPQ_TRY(rpq::fill_u64(oa.hist, kScores, 0, stream));
            hipLaunchKernelGGL(k_order_score, og, dim3(kBlock), 0, stream, oa);
            RPQ_LAUNCH_CHECK();
            RPQ_TRY(rpq::exclusive_scan_u64(oa.hist, oa.hist, kScores, oa.hist + kScores, nullptr, stream));
            hipLaunchKernelGGL(k_order_place, og, dim3(kBlock), 0, stream, oa);
            RPQ_LAUNCH_CHECK();
        }
        if (small) {
            hipLaunchKernelGGL(k_small_search, dim3(G_eff * (x.W / 32)), dim3(kSmallBlock), x.R * 8, stream, a,
                               x.max_len);
            RPQ_LAUNCH_CHECK();
        } else {
            // the bitmap's previous group must be extracted before it is cleared for this one
            if (side.stream && grp >= 2) RPQ_HIP(hipStreamWaitEvent(stream, side.extracted[buf], 0));
            RPQ_TRY(rpq::fill_u64(a.vis, G_eff * bitmap_words, 0, stream));
            if (x.seen_or) RPQ_TRY(rpq::fill_u64(a.ever, ((uint64_t)G_eff * x.R + 63) / 64, 0, stream));
            RPQ_TRY(rpq::fill_u64(reinterpret_cast<uint64_t*>(a.full), (G_eff * (uint64_t)x.R + 7) / 8, 0, stream));
            hipLaunchKernelGGL(k_seed, dim3((unsigned)(((uint64_t)G_eff * x.W + kBlock - 1) / kBlock)), dim3(kBlock), 0,
                               stream, a, G_eff, x.K);
            RPQ_LAUNCH_CHECK();
            const uint64_t n_rows = (uint64_t)G_eff * x.R;
            RPQ_DISPATCH_K(x.K, RPQ_TRY(launch_finalize<KK>(a, 0, n_rows, 0, x.max_len > 0, stream)));
            uint64_t level = 1;
            int p = 1;
            // a first-reach distance in the product graph is below Q * V, so the
            // fixpoint arrives within Q * V + 1 levels; more means a defect
            const uint64_t level_bound = (uint64_t)x.Q * x.V + 2;
            uint64_t launched = 0;
            // level l expands depth l - 1 and finalizes depth l; a length bound k stops after level k
            while (level <= x.max_len) {
                uint32_t n_launch = 0;
                for (; n_launch < x.sync_every && level <= x.max_len; ++n_launch) {
                    RPQ_DISPATCH_K(x.K, RPQ_TRY(launch_level<KK>(a, p, n_rows, (uint32_t)level, level < x.max_len,
                                                                  !noalloc, stream)));
                    p ^= 1;
                    ++level;
                }
                launched += n_launch;
                RPQ_HIP(hipMemcpyAsync(stage, a.counters, C_NCOUNTERS * 8, hipMemcpyDeviceToHost, stream));
                if (ps) RPQ_TRY(st.pump(false));   // the previous group's windows, while these levels run
                RPQ_HIP(hipStreamSynchronize(stream));
                if (!noalloc && profiler().on) profile_resolve();
                if (stage[C_ERR] & (ERR_LIST | ERR_DESC)) {
                    rpq::set_error("internal capacity exceeded (flags 0x%llx)", (unsigned long long)stage[C_ERR]);
                    return RPQ_EDEVICE;
                }
                if (stage[C_LIST + p] == 0) break;   // the last finalize produced no new entries
                if (launched > level_bound) {
                    rpq::set_error("no fixpoint after %llu levels", (unsigned long long)launched);
                    return RPQ_EDEVICE;
                }
            }
            if (launched == 0) {   // a bound of 0: only the seeds' zero-length walks
                RPQ_HIP(hipMemcpyAsync(stage, a.counters, C_NCOUNTERS * 8, hipMemcpyDeviceToHost, stream));
                RPQ_HIP(hipStreamSynchronize(stream));
            }
            const uint64_t lv = stage[C_LASTLEVEL];   // levels with a non-empty frontier, seeds included
            levels_total += lv;
            if (lv > 0 && lv - 1 > max_depth) max_depth = lv - 1;
        }
        if (side.stream) {
            RPQ_HIP(hipEventRecord(side.leveled, stream));
            RPQ_HIP(hipStreamWaitEvent(xs, side.leveled, 0));
        }
        // the previous group's windows read acc, partial and srcbase: all of them go on xs before
        // this group's count pass overwrites those arrays
        if (ps) RPQ_TRY(st.pump(true));
        if (tallies)
            RPQ_TRY(rpq::fill_u64(reinterpret_cast<uint64_t*>(ea.acc), (uint64_t)G_eff * x.W * 2, 0, xs));
        // profiling: the count pass timed on its own stream; it reads every final row of the group
        hipEvent_t xe0 = nullptr, xe1 = nullptr;
        if (!noalloc && profiler().on) {
            Profiler& pr = profiler();
            std::lock_guard<std::mutex> lk(pr.mu);
            xe0 = pr.get();
            xe1 = pr.get();
            pr.acc.extract_words += (uint64_t)G_eff * final_rows * x.K;
        }
        if (xe0) RPQ_HIP(hipEventRecord(xe0, xs));
        RPQ_DISPATCH_K(x.K, RPQ_TRY(launch_extract<KK>(a, tallies ? X_TALLIES : X_TOTALS, ea, xs)));
        if (xe0 && xe1) {
            RPQ_HIP(hipEventRecord(xe1, xs));
            Profiler& pr = profiler();
            std::lock_guard<std::mutex> lk(pr.mu);
            pr.pend_extract.emplace_back(xe0, xe1);
        }
        if (tallies) {
            const uint64_t n = (uint64_t)G_eff * x.W;
            uint64_t* per_source = (flags & RPQ_PER_SOURCE) ? res->per_source : nullptr;
            if (srcbase) {
                hipLaunchKernelGGL(k_chunk_prefix, dim3((unsigned)std::min<uint64_t>((n + kWaves - 1) / kWaves, 8192)),
                                   dim3(kBlock), 0, xs, ea.partial, n, x.nchunks);
                RPQ_LAUNCH_CHECK();
                hipLaunchKernelGGL((k_group_finish<true>), dim3(1), dim3(1024), 0, xs, a, ea.acc, srcbase, per_source,
                                   n);
            } else {
                hipLaunchKernelGGL((k_group_finish<false>), dim3((unsigned)((n + 1023) / 1024)), dim3(1024), 0, xs, a,
                                   ea.acc, srcbase, per_source, n);
            }
            RPQ_LAUNCH_CHECK();
        }
        if (want_pairs) {
            ea.pairs = res->pairs;
            ea.off = res->pair_offset;
            ea.cap = res->capacity;
            RPQ_DISPATCH_K(x.K, RPQ_TRY(launch_extract<KK>(a, X_KEYS, ea, xs)));
        }
        if (ps) {
            RPQ_TRY(st.start_group(a, ea, x.K, side.stream ? side.extracted[buf] : nullptr));
            RPQ_TRY(st.pump(false));
        } else if (side.stream) {
            RPQ_HIP(hipEventRecord(side.extracted[buf], xs));
        }
    }
    if (ps) RPQ_TRY(st.drain());
    if (side.stream) {
        // join: everything the side stream did happens before the totals are read on `stream`
        RPQ_HIP(hipEventRecord(side.leveled, xs));
        RPQ_HIP(hipStreamWaitEvent(stream, side.leveled, 0));
    }
    hipLaunchKernelGGL(k_tally_sum, dim3(1), dim3(1024), 0, stream, a.tally, a.xtally, a.counters);
    RPQ_LAUNCH_CHECK();
    RPQ_HIP(hipMemcpyAsync(stage, a.counters, C_NCOUNTERS * 8, hipMemcpyDeviceToHost, stream));
    RPQ_HIP(hipStreamSynchronize(stream));
    if (small) {
        levels_total = stage[C_LASTLEVEL];
        max_depth = levels_total ? levels_total - 1 : 0;
    }
    const uint64_t* const tally = stage + C_TALLY;
    if (!noalloc) {
        Profiler& pr = profiler();
        std::lock_guard<std::mutex> lk(pr.mu);
        if (pr.on) {
            pr.resolve(true);   // both streams are drained here
            pr.acc.finalize_rows += tally[T_FROWS];
            pr.acc.finalize_row_words += tally[T_FROWS] * x.K;
            pr.acc.finalize_words += tally[T_FWORDS];
            // 8-byte accesses of finalize to Vis: a read of every row word (seen OR), or a read and
            // a write of every non-zero word (two reads); less the reads of the second bitmap that rows
            // listed for the first time do without
            pr.acc.finalize_vis_words += x.seen_or ? (tally[T_FROWS] - tally[T_FFRESH]) * x.K : 2 * tally[T_FWORDS];
            // beyond the method's bytes: the Next word read beside each visited word (two reads);
            // seen OR makes the method's accesses only
            pr.acc.expand_extra_words += x.seen_or ? 0 : tally[T_WREAD];
            pr.acc.edge_items += tally[T_ITEMS];
            pr.acc.descriptors += tally[T_DESCS];
            pr.acc.row_words += tally[T_DESCS] * x.K;
            pr.acc.word_reads += tally[T_WREAD];
            pr.acc.word_updates += tally[T_WUPD];
        }
    }
    res->count = stage[C_COUNT];
    res->hash = stage[C_HASH];
    if (ps) res->written = st.delivered;
    res->product_edges = tally[T_EPROD];
    res->levels = levels_total;
    res->max_depth = max_depth;
    if (want_pairs) {
        const uint64_t avail = res->count > res->pair_offset ? res->count - res->pair_offset : 0;
        res->written = std::min<uint64_t>(avail, res->capacity);
        if (avail > res->capacity) {
            rpq::set_error("result has %llu keys past offset %llu; capacity is %llu",
                           (unsigned long long)avail, (unsigned long long)res->pair_offset,
                           (unsigned long long)res->capacity);
            return RPQ_EOVERFLOW;
        }
    }
    return RPQ_OK;
}

// Static scratch of the allocation-free entry point: a file-scope device array, one copy per
// device, held until the process ends.  In host code `scratch` only names the symbol; its device
// address comes from hipGetSymbolAddress, once per device, and only that address is used.
constexpr uint64_t kScratchBytes = RPQ_NOALLOC_SCRATCH_BYTES;
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

constexpr int kMaxDevices = 64;

void* scratch_address() {
    static std::mutex mu;
    static void* addr[kMaxDevices] = {};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) {
        rpq::set_error("no current HIP device (or device id beyond %d)", kMaxDevices - 1);
        return nullptr;
    }
    std::lock_guard<std::mutex> lk(mu);
    if (!addr[dev]) {
        void* p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p) {
            rpq::set_error("hipGetSymbolAddress(scratch) failed on device %d: %s", dev, hipGetErrorString(e));
            return nullptr;
        }
        addr[dev] = p;
    }
    return addr[dev];
}

}  // namespace

namespace rpq {

int eval_impl(rpq_graph_t g, const rpq_nfa* nfa, const uint32_t* sources, uint64_t n_sources, uint32_t flags,
              const rpq_eval_opts* opts, const uint64_t* target, void* workspace, uint64_t workspace_bytes,
              rpq_result* res, hipStream_t stream) {
    return eval_core(g, nfa, sources, n_sources, flags, opts, target, workspace, workspace_bytes, res, stream,
                     false);
}

}  // namespace rpq

extern "C" {

int rpq_eval_noalloc(rpq_graph_t g, const rpq_nfa* nfa, const uint32_t* sources, uint64_t n_sources,
                     uint32_t flags, const rpq_eval_opts* opts, rpq_result* res, hipStream_t stream) {
    rpq::clear_error();
    if (flags & RPQ_SPARSE) {
        rpq::set_error("rpq_eval_noalloc runs the bitmap search only; RPQ_SPARSE is not supported");
        return RPQ_EUNSUPPORTED;
    }
    if (!res) {
        rpq::set_error("result is NULL");
        return RPQ_EINVAL;
    }
    if ((flags & RPQ_LENGTH_BOUND) && !opts) {
        rpq::set_error("RPQ_LENGTH_BOUND needs opts->max_length");
        return RPQ_EINVAL;
    }
    uint64_t n = n_sources;
    if (g && (flags & RPQ_ALL_SOURCES) && n == 0) n = g->V;
    // the plan: the caller's knobs, with the unset ones narrowed until the workspace fits the
    // scratch (fewer units in flight first, then narrower units, then longer slices)
    rpq_eval_opts o{};
    if (opts) o = *opts;
    Plan plan;
    Layout lay;
    for (;;) {
        RPQ_TRY(prepare(g, nfa, n, flags, &o, &plan, &lay, true));
        if (lay.total <= kScratchBytes) break;
        if (!(opts && opts->concurrency) && lay.G > 1) {
            o.batch_width = lay.W;
            o.concurrency = lay.G / 2;
        } else if (!(opts && opts->batch_width) && lay.W > 64) {
            o.batch_width = lay.W / 2;
            o.concurrency = (opts && opts->concurrency) ? opts->concurrency : 0;
        } else if (!(opts && opts->chunk_edges) && lay.H < 4096) {
            o.batch_width = lay.W;
            o.concurrency = lay.G;
            o.chunk_edges = lay.H * 2;   // fewer slices
        } else {
            rpq::set_error("the evaluation needs %llu bytes of workspace; the static scratch holds %llu",
                           (unsigned long long)lay.total, (unsigned long long)kScratchBytes);
            res->workspace_needed = lay.total;
            return RPQ_ENOMEM;
        }
    }
    void* ws = scratch_address();
    if (!ws) return RPQ_EDEVICE;
    const int rc = eval_core(g, nfa, sources, n_sources, flags, &o, nullptr, ws, kScratchBytes, res, stream, true);
    if (rc != RPQ_OK && rc != RPQ_EOVERFLOW) (void)hipStreamSynchronize(stream);
    return rc;
}

int rpq_eval_stream(rpq_graph_t g, const rpq_nfa* nfa, const uint32_t* sources, uint64_t n_sources,
                    uint32_t flags, const rpq_eval_opts* opts, void* workspace, uint64_t workspace_bytes,
                    const rpq_pair_stream* out, rpq_result* res, hipStream_t stream) {
    rpq::clear_error();
    if (!out || !out->sink || !out->device_chunks || !out->host_chunks || out->chunk_keys == 0) {
        rpq::set_error("the pair stream needs a sink, two device and two host chunks of chunk_keys >= 1 keys");
        return RPQ_EINVAL;
    }
    if (flags & RPQ_SPARSE) {
        rpq::set_error("rpq_eval_stream runs the bitmap search only; RPQ_SPARSE is not supported");
        return RPQ_EUNSUPPORTED;
    }
    const int rc = eval_core(g, nfa, sources, n_sources, flags, opts, nullptr, workspace, workspace_bytes, res,
                             stream, false, out);
    if (rc != RPQ_OK) (void)hipStreamSynchronize(stream);
    return rc;
}

int rpq_profile_enable(int on) {
    Profiler& pr = profiler();
    std::lock_guard<std::mutex> lk(pr.mu);
    pr.on = on != 0;
    return RPQ_OK;
}

int rpq_profile_read(rpq_profile* out, int reset) {
    rpq::clear_error();
    if (!out) {
        rpq::set_error("out is NULL");
        return RPQ_EINVAL;
    }
    Profiler& pr = profiler();
    std::lock_guard<std::mutex> lk(pr.mu);
    *out = pr.acc;
    if (reset) pr.acc = rpq_profile{};
    return RPQ_OK;
}

}  // extern "C"
