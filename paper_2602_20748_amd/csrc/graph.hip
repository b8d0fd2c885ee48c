// Graph ingest: edge list -> label-partitioned CSR on the device.
//
// The paper keeps one adjacency per edge label (Labeled Grid Format,
// Section 2.4) so a traversal can follow exactly the edges an automaton
// transition asks for.  Here every (vertex, label) pair is one CSR row, rows
// ordered vertex-major so all label rows of a vertex share cache lines, and a
// per-vertex label bitmask lets the traversal skip labels with no edges.
//
// Steps (all on the device): pack (row, neighbour) into a uint64 key, stable
// radix sort, drop repeated keys (the edge relation is a set) and mark where
// each row starts, then fill the row pointers between the marks and derive the
// label masks from non-empty rows.  The in-edge CSR is the same construction
// with source and destination swapped.
//
// One scratch allocation serves both directions, each direction's arrays are
// one allocation, and released blocks are kept for the next graph (Blocks).
// The host waits once per direction.  How many edges are distinct is known only
// after the first direction: its neighbour array has room for all of the list
// until then, and is copied to a block of its size where much of it is unused.
#include "internal.h"

#include <algorithm>
#include <cstring>
#include <mutex>
#include <new>

namespace {

constexpr int kThreads = 256;

unsigned grid_for(uint64_t n, uint64_t cap = 65535) {
    uint64_t b = (n + kThreads - 1) / kThreads;
    if (b > cap) b = cap;
    return (unsigned)(b ? b : 1);
}

__global__ void k_make_keys(const uint32_t* __restrict__ a, const uint8_t* __restrict__ lab,
                            const uint32_t* __restrict__ b, uint64_t n, uint32_t V, uint32_t L,
                            uint64_t* __restrict__ keys, unsigned long long* __restrict__ err) {
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
        const uint32_t x = a[i], y = b[i], l = lab[i];
        if (x >= V || y >= V || l >= L) {
            atomicOr(err, 1ull);
            keys[i] = 0;
            continue;
        }
        keys[i] = ((uint64_t)(x * L + l) << 32) | y;
    }
}

// Keys (u, l, w) of one direction become (w, l, u) of the other.
__global__ void k_turn_keys(uint64_t* __restrict__ keys, uint64_t n, uint32_t L) {
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
        const uint64_t k = keys[i];
        const uint32_t row = (uint32_t)(k >> 32), u = row / L, l = row - u * L;
        keys[i] = ((uint64_t)((uint32_t)k * L + l) << 32) | u;
    }
}

// Distinct keys: a block takes kTile sorted keys; a first pass counts those that differ from their
// predecessor, a second writes them at the prefix of the counts and marks the start of each row.
constexpr uint32_t kTile = 2048;

__global__ __launch_bounds__(kThreads) void k_uniq_count(const uint64_t* __restrict__ keys, uint64_t n,
                                                         uint64_t* __restrict__ counts) {
    __shared__ uint32_t s_w[kThreads / 64];
    uint32_t c = 0;
    for (uint32_t j = threadIdx.x; j < kTile; j += kThreads) {
        const uint64_t i = (uint64_t)blockIdx.x * kTile + j;
        if (i < n && (i == 0 || keys[i] != keys[i - 1])) ++c;
    }
    c = (uint32_t)rpqd::wave_sum_u64(c);
    if ((threadIdx.x & 63) == 0) s_w[threadIdx.x >> 6] = c;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t t = 0;
        for (int w = 0; w < kThreads / 64; ++w) t += s_w[w];
        counts[blockIdx.x] = t;
    }
}

__global__ __launch_bounds__(kThreads) void k_uniq_write(const uint64_t* __restrict__ keys, uint64_t n,
                                                         const uint64_t* __restrict__ offs,
                                                         uint32_t* __restrict__ dst, uint32_t* __restrict__ start) {
    __shared__ uint32_t s_w[kThreads / 64];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    uint64_t at = offs[blockIdx.x];
    for (uint32_t j = threadIdx.x; j < kTile; j += kThreads) {
        const uint64_t i = (uint64_t)blockIdx.x * kTile + j;
        uint64_t k = 0, before = 0;
        bool first = false;
        if (i < n) {
            k = keys[i];
            before = i ? keys[i - 1] : ~k;
            first = k != before;
        }
        const uint64_t m = __ballot(first);
        if (lane == 0) s_w[wv] = (uint32_t)__popcll(m);
        __syncthreads();
        uint64_t pos = at + __popcll(m & rpqd::lanemask_lt());
        for (int w = 0; w < kThreads / 64; ++w) {
            pos += w < wv ? s_w[w] : 0;
            at += s_w[w];
        }
        if (first) {
            dst[pos] = (uint32_t)k;
            if ((k >> 32) != (before >> 32)) start[k >> 32] = (uint32_t)pos;
        }
        __syncthreads();
    }
}

// Row pointers from the marked starts (kNoRow: an empty row, which begins where the next one does).  A
// block takes kRows rows; what follows its last row comes from a suffix minimum over the blocks.
constexpr uint32_t kRows = 2048;
constexpr uint32_t kNoRow = 0xFFFFFFFFu;

__device__ __forceinline__ uint32_t wave_min_u32(uint32_t v) {
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) v = min(v, (uint32_t)__shfl_xor(v, o, 64));
    return v;
}

__global__ __launch_bounds__(kThreads) void k_row_min(const uint32_t* __restrict__ start, uint64_t R,
                                                      uint32_t* __restrict__ mins) {
    __shared__ uint32_t s_w[kThreads / 64];
    uint32_t m = kNoRow;
    for (uint32_t j = threadIdx.x; j < kRows; j += kThreads) {
        const uint64_t r = (uint64_t)blockIdx.x * kRows + j;
        if (r < R) m = min(m, start[r]);
    }
    m = wave_min_u32(m);
    if ((threadIdx.x & 63) == 0) s_w[threadIdx.x >> 6] = m;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 0; w < kThreads / 64; ++w) m = min(m, s_w[w]);
        mins[blockIdx.x] = m;
    }
}

// mins[b] = minimum over blocks after b, or the number of edges (one block, from the last entry down)
__global__ __launch_bounds__(1024) void k_row_after(uint32_t* __restrict__ mins, uint64_t nb,
                                                    const unsigned long long* __restrict__ n_edges) {
    __shared__ uint32_t s_w[16];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    uint32_t carry = (uint32_t)*n_edges;
    for (uint64_t top = nb; top > 0; top = top > 1024 ? top - 1024 : 0) {
        // thread t holds entry top - 1 - t: later blocks are lower threads
        const bool ok = threadIdx.x < top;
        const uint32_t x = ok ? mins[top - 1 - threadIdx.x] : kNoRow;
        uint32_t incl = x;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t y = __shfl_up(incl, o, 64);
            if (lane >= o) incl = min(incl, y);
        }
        if (lane == 63) s_w[wv] = incl;
        __syncthreads();
        uint32_t before = carry, all = carry;
        for (int w = 0; w < 16; ++w) {
            if (w < wv) before = min(before, s_w[w]);
            all = min(all, s_w[w]);
        }
        const uint32_t up = __shfl_up(incl, 1, 64);
        if (ok) mins[top - 1 - threadIdx.x] = lane ? min(before, up) : before;
        carry = all;
        __syncthreads();
    }
}

// In place: start becomes row_ptr[0 .. R].
__global__ __launch_bounds__(kThreads) void k_row_fill(uint32_t* __restrict__ row_ptr, uint64_t R,
                                                       const uint32_t* __restrict__ after,
                                                       const unsigned long long* __restrict__ n_edges) {
    constexpr uint32_t kEach = kRows / kThreads;   // consecutive rows of a thread
    static_assert(kEach == 8, "two 16-byte accesses");
    __shared__ uint32_t s_w[kThreads / 64];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const uint64_t r0 = (uint64_t)blockIdx.x * kRows + (uint64_t)threadIdx.x * kEach;
    uint4* const p4 = reinterpret_cast<uint4*>(row_ptr + r0);   // the array is 256-byte aligned
    const bool whole = r0 + kEach <= R;
    uint32_t x[kEach], lo = kNoRow;
    if (whole) {
        const uint4 u = p4[0], w = p4[1];
        x[0] = u.x, x[1] = u.y, x[2] = u.z, x[3] = u.w, x[4] = w.x, x[5] = w.y, x[6] = w.z, x[7] = w.w;
    } else {
#pragma unroll
        for (uint32_t j = 0; j < kEach; ++j) x[j] = r0 + j < R ? row_ptr[r0 + j] : kNoRow;
    }
#pragma unroll
    for (uint32_t j = 0; j < kEach; ++j) lo = min(lo, x[j]);
    // minimum over the threads after this one
    uint32_t incl = lo;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t y = __shfl_down(incl, o, 64);
        if (lane + o < 64) incl = min(incl, y);
    }
    if (lane == 0) s_w[wv] = incl;
    __syncthreads();
    uint32_t next = after[blockIdx.x];
    for (int w = wv + 1; w < kThreads / 64; ++w) next = min(next, s_w[w]);
    const uint32_t later = __shfl_down(incl, 1, 64);
    if (lane < 63) next = min(next, later);
#pragma unroll
    for (int j = kEach - 1; j >= 0; --j) x[j] = next = min(next, x[j]);   // starts ascend
    if (whole) {
        p4[0] = make_uint4(x[0], x[1], x[2], x[3]);
        p4[1] = make_uint4(x[4], x[5], x[6], x[7]);
    } else {
        for (uint32_t j = 0; j < kEach; ++j)
            if (r0 + j < R) row_ptr[r0 + j] = x[j];
    }
    if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) row_ptr[R] = (uint32_t)*n_edges;
}

// Label masks of the vertices; edges per label and rows with edges.  A wave's 64 vertices have 64 L rows, lane
// + 64 t in step t, so a lane meets the same label in the same step of every wave and adds its edges into a
// word of its own per step (one counter per label instead: 64 lanes on a few addresses, 112 us at 8M rows).
__global__ __launch_bounds__(kThreads) void k_label_mask(const uint32_t* __restrict__ row_ptr, uint32_t V, uint32_t L,
                                                         uint64_t* __restrict__ lmask,
                                                         unsigned long long* __restrict__ per_label,
                                                         unsigned long long* __restrict__ nonempty) {
    extern __shared__ uint32_t s_edges[];   // [L][64]
    __shared__ unsigned long long s_m[kThreads / 64][64];
    __shared__ uint32_t s_lab[RPQ_MAX_LABELS];
    __shared__ uint32_t s_rows;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    for (uint32_t i = threadIdx.x; i < 64 * L; i += kThreads) s_edges[i] = 0;
    for (uint32_t i = threadIdx.x; i < L; i += kThreads) s_lab[i] = 0;
    if (threadIdx.x == 0) s_rows = 0;
    __syncthreads();
    const uint64_t stride = (uint64_t)gridDim.x * (kThreads / 64);
    const uint32_t v_step = 64 / L, l_step = 64 % L, v_first = lane / L, l_first = lane % L;
    uint32_t rows = 0;
    for (uint64_t w = (uint64_t)blockIdx.x * (kThreads / 64) + wv; w * 64 < V; w += stride) {
        s_m[wv][lane] = 0;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        const uint64_t r0 = w * 64 * L;
        const uint32_t n = (uint32_t)min((uint64_t)64, V - w * 64) * L;
        uint32_t v = v_first, l = l_first;
        for (uint32_t i = lane; i < n; i += 64) {
            const uint32_t d = row_ptr[r0 + i + 1] - row_ptr[r0 + i];
            if (d) {
                atomicOr(&s_m[wv][v], 1ull << l);
                atomicAdd(&s_edges[i], d);
                ++rows;
            }
            v += v_step;
            l += l_step;
            if (l >= L) {
                l -= L;
                ++v;
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        if (w * 64 + lane < V) lmask[w * 64 + lane] = s_m[wv][lane];
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }
    rows = (uint32_t)rpqd::wave_sum_u64(rows);
    if (lane == 0 && rows) atomicAdd(&s_rows, rows);
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < 64 * L; i += kThreads)
        if (s_edges[i]) atomicAdd(&s_lab[i % L], s_edges[i]);
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < L; i += kThreads)
        if (s_lab[i]) atomicAdd(&per_label[i], (unsigned long long)s_lab[i]);
    if (threadIdx.x == 0 && s_rows) atomicAdd(nonempty, (unsigned long long)s_rows);
}

// entered bits of a direction, from its keys (row << 32 | neighbour).  Hubs are entered by many edges: a
// bit that is already set is not ORed again.
__global__ void k_entered(const uint64_t* __restrict__ keys, uint64_t m, uint32_t L, uint64_t n_words,
                          unsigned long long* __restrict__ entered) {
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < m; i += stride) {
        const uint64_t k = keys[i];
        const uint32_t v = (uint32_t)k;
        unsigned long long* w = &entered[(uint64_t)((uint32_t)(k >> 32) % L) * n_words + (v >> 6)];
        const unsigned long long bit = 1ull << (v & 63);
        if (!(*w & bit)) atomicOr(w, bit);
    }
}

// the same from the other direction's label masks: v is entered by the labels it leaves by there
__global__ void k_entered_from_masks(const uint64_t* __restrict__ lmask, uint32_t V, uint32_t L, uint64_t n_words,
                                     uint64_t* __restrict__ entered) {
    const int lane = threadIdx.x & 63;
    const uint64_t stride = (uint64_t)gridDim.x * (blockDim.x / 64);
    for (uint64_t w = (uint64_t)blockIdx.x * (blockDim.x / 64) + (threadIdx.x >> 6); w < n_words; w += stride) {
        const uint64_t v = w * 64 + lane;
        const uint64_t m = v < V ? lmask[v] : 0;
        for (uint32_t l = 0; l < L; ++l) {
            const uint64_t b = __ballot((m >> l) & 1);
            if (lane == 0) entered[(uint64_t)l * n_words + w] = b;
        }
    }
}

// counts[l] += bits of entered[l]; one block row (gridDim.y) per label
__global__ void k_entered_counts(const uint64_t* __restrict__ entered, uint64_t n_words,
                                 unsigned long long* __restrict__ counts) {
    uint64_t c = 0;
    const uint64_t* e = entered + (uint64_t)blockIdx.y * n_words;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n_words;
         i += (uint64_t)gridDim.x * blockDim.x)
        c += __popcll(e[i]);
    c = rpqd::wave_sum_u64(c);
    if ((threadIdx.x & 63) == 0 && c) atomicAdd(&counts[blockIdx.y], (unsigned long long)c);
}

// Device memory of graphs and their builds.  The runtime takes 0.25 ms to release a block, and 15 ms and more
// each while it is still clearing much other memory released shortly before: a build of 16M edges both ways
// then took 45 ms, of which its kernels were 2, and takes 1.75 ms with its blocks kept.  So up to kKept bytes in
// kSlots released blocks wait for the next build.  That is the end of the gain: the scratch alone, 16 bytes an
// edge, passes kKept from 2^26 edges on, and such a build takes and releases its memory each time (2^22
// vertices, 2^26 edges both ways: 8.4 ms; 20.8 when nothing was kept and the kernels took longer).  A block
// comes here only when no work uses it any more, so any stream may take it; it goes back to the runtime when a
// newer block needs its room, when two builds in a row had no use for it, or when an allocation here fails.
// Sizes are rounded up to a sixteenth of their power of two, and a kept block serves only its own size: what a
// graph holds does not depend on what was released before it.
class Blocks {
public:
    static constexpr uint64_t kKept = 1ull << 30;
    static constexpr int kSlots = 16;

    static uint64_t rounded(uint64_t bytes) {
        uint64_t step = 256;
        while (step * 32 <= bytes) step *= 2;
        return (std::max<uint64_t>(1, bytes) + step - 1) / step * step;
    }

    int take(uint64_t bytes, rpq::Block* out) {
        bytes = rounded(bytes);
        int dev = 0;
        (void)hipGetDevice(&dev);
        {
            std::lock_guard<std::mutex> lk(mu_);
            for (int i = 0; i < n_; ++i)
                if (kept_[i].b.device == dev && kept_[i].b.bytes == bytes) {
                    *out = drop(i);
                    return RPQ_OK;
                }
        }
        hipError_t e = hipMalloc(&out->p, bytes);
        if (e == hipErrorOutOfMemory && let_go([](const Kept&) { return true; })) {
            (void)hipGetLastError();
            e = hipMalloc(&out->p, bytes);
        }
        if (e != hipSuccess) {
            (void)hipGetLastError();
            *out = rpq::Block();
            rpq::set_error("hipMalloc(%llu) failed: %s", (unsigned long long)bytes, hipGetErrorString(e));
            return e == hipErrorOutOfMemory ? RPQ_ENOMEM : RPQ_EDEVICE;
        }
        out->bytes = bytes;
        out->device = dev;
        return RPQ_OK;
    }
    // idle: the caller has waited for everything on the current device that used the block
    void give(rpq::Block* b, bool idle) {
        if (!b->p) return;
        int dev = -1;
        (void)hipGetDevice(&dev);
        rpq::Block gone[kSlots + 1];
        int n_gone = 0;
        if (idle && b->device == dev && b->bytes <= kKept) {
            std::lock_guard<std::mutex> lk(mu_);
            while (n_ == kSlots || total_ + b->bytes > kKept) gone[n_gone++] = drop(0);   // oldest first
            kept_[n_++] = {*b, builds_};
            total_ += b->bytes;
        } else {
            gone[n_gone++] = *b;
        }
        for (int i = 0; i < n_gone; ++i) (void)hipFree(gone[i].p);
        *b = rpq::Block();
    }
    void build_begins() {
        uint64_t now;
        {
            std::lock_guard<std::mutex> lk(mu_);
            now = ++builds_;
        }
        let_go([now](const Kept& k) { return now > k.since + 2; });
    }

private:
    struct Kept {
        rpq::Block b;
        uint64_t since;   // builds begun when it came
    };
    rpq::Block drop(int i) {
        const rpq::Block b = kept_[i].b;
        total_ -= b.bytes;
        for (--n_; i < n_; ++i) kept_[i] = kept_[i + 1];
        return b;
    }
    // The blocks that `which` names go back to the runtime, which may wait for the device: outside the lock, so
    // that a build on another thread does not wait too.  Returns whether there were any.
    template <class F>
    bool let_go(F which) {
        rpq::Block gone[kSlots];
        int n_gone = 0;
        {
            std::lock_guard<std::mutex> lk(mu_);
            for (int i = n_; i-- > 0;)
                if (which(kept_[i])) gone[n_gone++] = drop(i);
        }
        for (int i = 0; i < n_gone; ++i) (void)hipFree(gone[i].p);
        return n_gone > 0;
    }
    std::mutex mu_;
    Kept kept_[kSlots];
    int n_ = 0;
    uint64_t total_ = 0, builds_ = 0;
};

Blocks& blocks() {
    static Blocks* b = new Blocks();   // outlives every graph; what it still holds goes with the process
    return *b;
}

// Scratch of a build: the keys and their sorting, shared by the two directions.
struct Scratch {
    rpq::Block mem, old;   // old: a block that the build moved out of
    hipStream_t stream;
    explicit Scratch(hipStream_t s) : stream(s) {}
    ~Scratch() {
        const bool idle = hipStreamSynchronize(stream) == hipSuccess;   // a failed build may leave work queued
        blocks().give(&old, idle);
        blocks().give(&mem, idle);
    }
    Scratch(const Scratch&) = delete;
    Scratch& operator=(const Scratch&) = delete;
    uint64_t *keys, *alt, *sorted, *counts, *scan;   // sorted: the one of the two that holds the keys
    uint32_t* mins;
    void* sort;
    unsigned long long* ctr;   // [kCtr]

    static constexpr uint64_t kCtr = 4 + 3 * RPQ_MAX_LABELS;

    int alloc(uint64_t n_edges, uint64_t R) {
        const uint64_t tiles = (n_edges + kTile - 1) / kTile + 1;
        uint64_t off = 0;
        auto take = [&](uint64_t bytes) {
            const uint64_t o = off;
            off += (bytes + 255) / 256 * 256;
            return o;
        };
        const uint64_t o_keys = take(n_edges * 8), o_alt = take(n_edges * 8), o_counts = take(tiles * 8),
                       o_scan = take((rpq::scan_temp_elems(tiles) + 1) * 8),
                       o_mins = take(((R + kRows - 1) / kRows) * 4), o_sort = take(rpq::radix_temp_bytes(n_edges)),
                       o_ctr = take(kCtr * 8);
        RPQ_TRY(blocks().take(off, &mem));
        char* b = reinterpret_cast<char*>(mem.p);
        keys = sorted = reinterpret_cast<uint64_t*>(b + o_keys);
        alt = reinterpret_cast<uint64_t*>(b + o_alt);
        counts = reinterpret_cast<uint64_t*>(b + o_counts);
        scan = reinterpret_cast<uint64_t*>(b + o_scan);
        mins = reinterpret_cast<uint32_t*>(b + o_mins);
        sort = b + o_sort;
        ctr = reinterpret_cast<unsigned long long*>(b + o_ctr);
        return RPQ_OK;
    }
};

// Bytes of a direction's arrays with room for n_dst neighbours, which come last; out's pointers where mem is set.
uint64_t place_csr(uint32_t V, uint32_t L, uint64_t n_dst, rpq::Csr* out) {
    auto up = [](uint64_t x) { return (x + 255) / 256 * 256; };
    const uint64_t o_mask = up(((uint64_t)V * L + 1) * 4), o_ent = o_mask + up((uint64_t)V * 8),
                   o_dst = o_ent + up(L * (((uint64_t)V + 63) / 64) * 8);
    if (char* mem = reinterpret_cast<char*>(out->mem.p)) {
        out->row_ptr = reinterpret_cast<uint32_t*>(mem);
        out->lmask = reinterpret_cast<uint64_t*>(mem + o_mask);
        out->entered = reinterpret_cast<uint64_t*>(mem + o_ent);
        out->dst = reinterpret_cast<uint32_t*>(mem + o_dst);
    }
    return o_dst + std::max<uint64_t>(1, n_dst) * 4;
}

// Moves a direction to a block with room for its E neighbours alone, if there is one.  The old block is in use
// until the stream has copied it: it goes with the scratch.
int trim_csr(uint32_t V, uint32_t L, uint64_t E, Scratch& sc, rpq::Csr* out, hipStream_t s) {
    rpq::Csr t;
    const uint64_t bytes = place_csr(V, L, E, &t);
    if (blocks().take(bytes, &t.mem) != RPQ_OK) {
        rpq::clear_error();
        return RPQ_OK;
    }
    sc.old = out->mem;
    out->mem = t.mem;
    place_csr(V, L, E, out);
    RPQ_HIP(hipMemcpyAsync(out->mem.p, sc.old.p, bytes, hipMemcpyDeviceToDevice, s));
    return RPQ_OK;
}

// Build one CSR direction (more: the other one follows).  a/b: row-side and neighbour-side endpoint arrays.
// n_dst: room for its distinct edges.  other: the direction built before this one (its label masks then give
// this one's entered bits, and this one's give its), or null.
int build_csr(const uint32_t* a, const uint8_t* lab, const uint32_t* b, uint64_t n_edges, uint64_t n_dst, uint32_t V,
              uint32_t L, Scratch& sc, rpq::Csr* out, rpq::Csr* other, bool more, uint64_t* E_out,
              uint64_t* per_label, uint64_t* stage, hipStream_t s) {
    using namespace rpq;
    const uint64_t R = (uint64_t)V * L;
    const uint64_t n_words = ((uint64_t)V + 63) / 64;
    RPQ_TRY(blocks().take(place_csr(V, L, n_dst, out), &out->mem));
    place_csr(V, L, n_dst, out);
    unsigned long long* c = sc.ctr;   // [0] err [1] distinct edges [2] nonempty rows
    unsigned long long* pl = c + 4;
    unsigned long long* ent = pl + RPQ_MAX_LABELS;   // [2][RPQ_MAX_LABELS]: entered counts, this and other
    RPQ_TRY(fill_u64(reinterpret_cast<uint64_t*>(c), Scratch::kCtr, 0, s));
    RPQ_TRY(fill_u32(out->row_ptr, R + 1, kNoRow, s));
    uint64_t* sorted = sc.sorted;
    if (n_edges) {
        // The first direction's sorted keys are in the order of u, so the second's take a stable sort by row
        // alone: three passes instead of six at 2^20 vertices and 8 labels (16M edges: 1.06 -> 0.63 ms).  In
        // the first, an edge outside the graph becomes key 0 and an error below.
        if (other)
            hipLaunchKernelGGL(k_turn_keys, dim3(grid_for(n_edges)), dim3(kThreads), 0, s, sorted, n_edges, L);
        else
            hipLaunchKernelGGL(k_make_keys, dim3(grid_for(n_edges)), dim3(kThreads), 0, s, a, lab, b, n_edges, V, L,
                               sorted, c);
        RPQ_LAUNCH_CHECK();
        RPQ_TRY(radix_sort_u64(sorted, sorted == sc.keys ? sc.alt : sc.keys, n_edges,
                               other ? 0 : bits_for(V ? V - 1 : 0), bits_for(R ? R - 1 : 0), sc.sort, s, &sorted));
        sc.sorted = sorted;
        const uint64_t tiles = (n_edges + kTile - 1) / kTile;
        hipLaunchKernelGGL(k_uniq_count, dim3((unsigned)tiles), dim3(kThreads), 0, s, sorted, n_edges, sc.counts);
        RPQ_LAUNCH_CHECK();
        RPQ_TRY(exclusive_scan_u64(sc.counts, sc.counts, tiles, sc.scan, reinterpret_cast<uint64_t*>(c + 1), s));
        hipLaunchKernelGGL(k_uniq_write, dim3((unsigned)tiles), dim3(kThreads), 0, s, sorted, n_edges, sc.counts,
                           out->dst, out->row_ptr);
        RPQ_LAUNCH_CHECK();
    }
    const uint64_t rblocks = (R + kRows - 1) / kRows;
    hipLaunchKernelGGL(k_row_min, dim3((unsigned)rblocks), dim3(kThreads), 0, s, out->row_ptr, R, sc.mins);
    RPQ_LAUNCH_CHECK();
    hipLaunchKernelGGL(k_row_after, dim3(1), dim3(1024), 0, s, sc.mins, rblocks, c + 1);
    RPQ_LAUNCH_CHECK();
    hipLaunchKernelGGL(k_row_fill, dim3((unsigned)rblocks), dim3(kThreads), 0, s, out->row_ptr, R, sc.mins, c + 1);
    RPQ_LAUNCH_CHECK();
    hipLaunchKernelGGL(k_label_mask, dim3(grid_for(n_words * 64, 1024)), dim3(kThreads), L * 256, s, out->row_ptr, V,
                       L, out->lmask, pl, c + 2);
    RPQ_LAUNCH_CHECK();
    // entered bits: for both directions from the other's masks once both are there, else from the edges
    const dim3 cgrid(grid_for(n_words, 32), L);
    for (int i = 0; i < 2; ++i) {
        rpq::Csr* t = i == 0 ? out : other;
        if (!t || (i == 0 && more)) continue;
        if (other) {
            hipLaunchKernelGGL(k_entered_from_masks, dim3(grid_for(n_words * 64, 4096)), dim3(kThreads), 0, s,
                               i == 0 ? other->lmask : out->lmask, V, L, n_words, t->entered);
        } else {
            RPQ_TRY(fill_u64(t->entered, L * n_words, 0, s));
            hipLaunchKernelGGL(k_entered, dim3(grid_for(n_edges, 8192)), dim3(kThreads), 0, s, sorted, n_edges, L,
                               n_words, reinterpret_cast<unsigned long long*>(t->entered));
        }
        RPQ_LAUNCH_CHECK();
        hipLaunchKernelGGL(k_entered_counts, cgrid, dim3(kThreads), 0, s, t->entered, n_words,
                           ent + i * RPQ_MAX_LABELS);
        RPQ_LAUNCH_CHECK();
    }
    RPQ_HIP(hipMemcpyAsync(stage, c, Scratch::kCtr * 8, hipMemcpyDeviceToHost, s));
    RPQ_HIP(hipStreamSynchronize(s));
    if (stage[0]) {
        set_error("edge list holds a vertex id >= n_vertices or a label id >= n_labels");
        return RPQ_EINVAL;
    }
    if (stage[1] >= 0xFFFFFFFFull) {
        set_error("more than 2^32-1 distinct edges");
        return RPQ_EUNSUPPORTED;
    }
    out->nonempty_rows = stage[2];
    if (per_label)
        for (uint32_t l = 0; l < L; ++l) per_label[l] = stage[4 + l];
    for (uint32_t l = 0; l < L; ++l) {
        out->n_entered[l] = stage[4 + RPQ_MAX_LABELS + l];
        if (other) other->n_entered[l] = stage[4 + 2 * RPQ_MAX_LABELS + l];
    }
    *E_out = stage[1];
    return RPQ_OK;
}

void free_graph(rpq_graph* g) {
    if (!g) return;
    const bool idle = hipDeviceSynchronize() == hipSuccess;
    blocks().give(&g->out.mem, idle);
    blocks().give(&g->in.mem, idle);
    blocks().give(&g->vlabels, idle);
    delete g;
}

}  // namespace

extern "C" {

int rpq_graph_create(const uint32_t* src, const uint8_t* label, const uint32_t* dst, uint64_t n_edges,
                     uint32_t n_vertices, uint32_t n_labels, const uint8_t* vertex_label, uint32_t flags,
                     hipStream_t stream, rpq_graph_t* out) {
    rpq::clear_error();
    if (!out) {
        rpq::set_error("out is NULL");
        return RPQ_EINVAL;
    }
    *out = nullptr;
    if (n_vertices == 0 || n_vertices > (1u << 31)) {
        rpq::set_error("n_vertices must be in [1, 2^31]");
        return RPQ_EINVAL;
    }
    if (n_labels == 0 || n_labels > RPQ_MAX_LABELS) {
        rpq::set_error("n_labels must be in [1, %d]", RPQ_MAX_LABELS);
        return RPQ_EINVAL;
    }
    if ((uint64_t)n_vertices * n_labels >= 0xFFFFFFFFull) {
        rpq::set_error("n_vertices * n_labels must be below 2^32");
        return RPQ_EINVAL;
    }
    if (n_edges && (!src || !label || !dst)) {
        rpq::set_error("edge arrays are NULL");
        return RPQ_EINVAL;
    }
    if (flags & ~RPQ_BUILD_IN_CSR) {
        rpq::set_error("unknown flags 0x%x", flags);
        return RPQ_EINVAL;
    }
    rpq_graph* g = new (std::nothrow) rpq_graph();
    if (!g) {
        rpq::set_error("host allocation failed");
        return RPQ_ENOMEM;
    }
    g->V = n_vertices;
    g->L = n_labels;
    g->E_in = n_edges;
    uint64_t* stage = rpq::host_stage();
    if (hipGetDevice(&g->device) != hipSuccess || !stage) {
        rpq::set_error("HIP device or pinned staging unavailable");
        free_graph(g);
        return RPQ_EDEVICE;
    }
    const bool both = (flags & RPQ_BUILD_IN_CSR) != 0;
    blocks().build_begins();
    Scratch sc(stream);
    int rc = sc.alloc(n_edges, (uint64_t)n_vertices * n_labels);
    if (rc == RPQ_OK)
        rc = build_csr(src, label, dst, n_edges, n_edges, n_vertices, n_labels, sc, &g->out, nullptr, both, &g->E,
                       g->per_label, stage, stream);
    // a copy of what is used costs less than a sixteenth of the build (16M edges: 25 us of 1.75 ms)
    if (rc == RPQ_OK && (n_edges - g->E) * 4 > g->out.mem.bytes / 16)
        rc = trim_csr(n_vertices, n_labels, g->E, sc, &g->out, stream);
    if (rc == RPQ_OK && both) {
        uint64_t e_in = 0;
        rc = build_csr(dst, label, src, n_edges, g->E, n_vertices, n_labels, sc, &g->in, &g->out, false, &e_in,
                       nullptr, stage, stream);
        g->has_in = rc == RPQ_OK;
    }
    if (rc == RPQ_OK && vertex_label) {
        rc = blocks().take(n_vertices, &g->vlabels);
        if (rc == RPQ_OK) {
            g->vlabel = reinterpret_cast<uint8_t*>(g->vlabels.p);
            if (hipMemcpyAsync(g->vlabel, vertex_label, n_vertices, hipMemcpyDeviceToDevice, stream) != hipSuccess ||
                hipStreamSynchronize(stream) != hipSuccess) {
                rpq::set_error("copying vertex labels failed");
                rc = RPQ_EDEVICE;
            }
        }
    }
    if (rc != RPQ_OK) {
        free_graph(g);
        return rc;
    }
    g->device_bytes = g->out.mem.bytes + g->in.mem.bytes + g->vlabels.bytes;
    *out = g;
    return RPQ_OK;
}

int rpq_graph_destroy(rpq_graph_t g) {
    if (!g) return RPQ_OK;
    free_graph(g);
    return RPQ_OK;
}

int rpq_graph_info_get(rpq_graph_t g, rpq_graph_info* out) {
    rpq::clear_error();
    if (!g || !out) {
        rpq::set_error("NULL argument");
        return RPQ_EINVAL;
    }
    std::memset(out, 0, sizeof *out);
    out->n_vertices = g->V;
    out->n_labels = g->L;
    out->n_edges_in = g->E_in;
    out->n_edges = g->E;
    for (uint32_t l = 0; l < g->L; ++l) out->edges_per_label[l] = g->per_label[l];
    out->nonempty_rows = g->out.nonempty_rows;
    out->device_bytes = g->device_bytes;
    out->has_in_csr = g->has_in ? 1 : 0;
    out->has_vertex_labels = g->vlabel ? 1 : 0;
    return RPQ_OK;
}

int rpq_graph_export_csr(rpq_graph_t g, int reverse, uint32_t* row_ptr, uint32_t* dst, hipStream_t stream) {
    rpq::clear_error();
    if (!g) {
        rpq::set_error("NULL graph");
        return RPQ_EINVAL;
    }
    const rpq::Csr& c = reverse ? g->in : g->out;
    if (reverse && !g->has_in) {
        rpq::set_error("graph has no in-edge CSR");
        return RPQ_EUNSUPPORTED;
    }
    const uint64_t R = (uint64_t)g->V * g->L;
    if (row_ptr) RPQ_HIP(hipMemcpyAsync(row_ptr, c.row_ptr, (R + 1) * 4, hipMemcpyDeviceToDevice, stream));
    if (dst && g->E) RPQ_HIP(hipMemcpyAsync(dst, c.dst, g->E * 4, hipMemcpyDeviceToDevice, stream));
    RPQ_HIP(hipStreamSynchronize(stream));
    return RPQ_OK;
}

}  // extern "C"
