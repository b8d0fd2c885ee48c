// Device-wide primitives used by graph ingest and the join: fills, an
// exclusive scan over uint64 and a stable LSD radix sort of uint64 keys.
//
// The sort ranks equal digits inside a wave64 by matching the 8 digit bits
// with 8 ballots (lanes whose digit agrees on every bit form a group); blocks
// take contiguous tiles and use no global atomics, so the order of equal
// digits is preserved across the grid.
#include "internal.h"

#include <cstdarg>
#include <cstring>
#include <string>

namespace rpq {

// ------------------------------------------------------------------------------------------------
// errors (thread-local message)
// ------------------------------------------------------------------------------------------------
static thread_local std::string g_last_error;

void set_error(const char* fmt, ...) {
    char buf[1024];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    g_last_error = buf;
}

void clear_error() { g_last_error.clear(); }

const char* last_error_cstr() { return g_last_error.c_str(); }

// ------------------------------------------------------------------------------------------------
// fills
// ------------------------------------------------------------------------------------------------
__global__ void k_fill_u64(uint64_t* __restrict__ p, uint64_t n, uint64_t value) {
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    // two-word stores where the pointer allows it
    if ((reinterpret_cast<uintptr_t>(p) & 15) == 0) {
        ulonglong2* p2 = reinterpret_cast<ulonglong2*>(p);
        const uint64_t n2 = n / 2;
        for (uint64_t j = i; j < n2; j += stride) p2[j] = make_ulonglong2(value, value);
        if (i == 0 && (n & 1)) p[n - 1] = value;
    } else {
        for (uint64_t j = i; j < n; j += stride) p[j] = value;
    }
}

__global__ void k_fill_u32(uint32_t* __restrict__ p, uint64_t n, uint32_t value) {
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) p[i] = value;
}

static unsigned fill_grid(uint64_t n) {
    uint64_t b = (n + 255) / 256;
    if (b > 8192) b = 8192;
    if (b == 0) b = 1;
    return (unsigned)b;
}

int fill_u64(uint64_t* p, uint64_t n, uint64_t value, hipStream_t s) {
    if (n == 0) return RPQ_OK;
    hipLaunchKernelGGL(k_fill_u64, dim3(fill_grid(n / 2 + 1)), dim3(256), 0, s, p, n, value);
    RPQ_LAUNCH_CHECK();
    return RPQ_OK;
}

int fill_u32(uint32_t* p, uint64_t n, uint32_t value, hipStream_t s) {
    if (n == 0) return RPQ_OK;
    hipLaunchKernelGGL(k_fill_u32, dim3(fill_grid(n)), dim3(256), 0, s, p, n, value);
    RPQ_LAUNCH_CHECK();
    return RPQ_OK;
}

// ------------------------------------------------------------------------------------------------
// exclusive scan (uint64), 1024 elements per 256-thread block, recursive over block sums
// ------------------------------------------------------------------------------------------------
constexpr int kScanThreads = 256;
constexpr int kScanItems = 4;
constexpr uint64_t kScanTile = kScanThreads * kScanItems;

__global__ __launch_bounds__(kScanThreads) void k_scan_reduce(const uint64_t* __restrict__ in, uint64_t n,
                                                              uint64_t* __restrict__ sums) {
    __shared__ uint64_t s_w[kScanThreads / 64];
    const uint64_t base = (uint64_t)blockIdx.x * kScanTile + (uint64_t)threadIdx.x * kScanItems;
    uint64_t t = 0;
#pragma unroll
    for (int i = 0; i < kScanItems; ++i)
        if (base + i < n) t += in[base + i];
    t = rpqd::wave_sum_u64(t);
    if ((threadIdx.x & 63) == 0) s_w[threadIdx.x >> 6] = t;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint64_t s = 0;
        for (int w = 0; w < kScanThreads / 64; ++w) s += s_w[w];
        sums[blockIdx.x] = s;
    }
}

__global__ __launch_bounds__(kScanThreads) void k_scan_apply(const uint64_t* in, uint64_t* out, uint64_t n,
                                                             const uint64_t* __restrict__ offsets,
                                                             uint64_t* __restrict__ total) {
    __shared__ uint64_t s_w[kScanThreads / 64];
    const uint64_t base = (uint64_t)blockIdx.x * kScanTile + (uint64_t)threadIdx.x * kScanItems;
    uint64_t v[kScanItems];
    uint64_t t = 0;
#pragma unroll
    for (int i = 0; i < kScanItems; ++i) {
        v[i] = (base + i < n) ? in[base + i] : 0;
        t += v[i];
    }
    const uint64_t incl = rpqd::wave_incl_scan_u64(t);
    const int wv = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 63) s_w[wv] = incl;
    __syncthreads();
    uint64_t pre = offsets ? offsets[blockIdx.x] : 0;
    for (int w = 0; w < wv; ++w) pre += s_w[w];
    uint64_t run = pre + incl - t;
#pragma unroll
    for (int i = 0; i < kScanItems; ++i) {
        if (base + i < n) out[base + i] = run;
        run += v[i];
    }
    if (total && blockIdx.x == gridDim.x - 1 && threadIdx.x == kScanThreads - 1) *total = run;
}

uint64_t scan_temp_elems(uint64_t n) {
    const uint64_t nb = (n + kScanTile - 1) / kScanTile;
    if (nb <= 1) return 0;
    return nb + scan_temp_elems(nb);
}

int exclusive_scan_u64(const uint64_t* in, uint64_t* out, uint64_t n, uint64_t* temp, uint64_t* total,
                       hipStream_t s) {
    if (n == 0) {
        if (total) RPQ_TRY(fill_u64(total, 1, 0, s));
        return RPQ_OK;
    }
    const uint64_t nb = (n + kScanTile - 1) / kScanTile;
    if (nb == 1) {
        hipLaunchKernelGGL(k_scan_apply, dim3(1), dim3(kScanThreads), 0, s, in, out, n, nullptr, total);
        RPQ_LAUNCH_CHECK();
        return RPQ_OK;
    }
    uint64_t* sums = temp;
    hipLaunchKernelGGL(k_scan_reduce, dim3((unsigned)nb), dim3(kScanThreads), 0, s, in, n, sums);
    RPQ_LAUNCH_CHECK();
    RPQ_TRY(exclusive_scan_u64(sums, sums, nb, temp + nb, nullptr, s));
    hipLaunchKernelGGL(k_scan_apply, dim3((unsigned)nb), dim3(kScanThreads), 0, s, in, out, n, sums, total);
    RPQ_LAUNCH_CHECK();
    return RPQ_OK;
}

// ------------------------------------------------------------------------------------------------
// stable LSD radix sort, 8-bit digits
// ------------------------------------------------------------------------------------------------
constexpr int kSortThreads = 256;
constexpr int kSortWaves = kSortThreads / 64;
constexpr int kSortKeys = 16;                           // keys per thread
constexpr uint64_t kSortTile = (uint64_t)kSortThreads * kSortKeys;

__global__ __launch_bounds__(kSortThreads) void k_radix_hist(const uint64_t* __restrict__ keys, uint64_t n,
                                                             int shift, uint64_t* __restrict__ hist,
                                                             uint32_t nb) {
    __shared__ uint32_t cnt[256];
    cnt[threadIdx.x] = 0;
    __syncthreads();
    const uint64_t base = (uint64_t)blockIdx.x * kSortTile;
    for (int c = 0; c < kSortKeys; ++c) {
        const uint64_t i = base + (uint64_t)c * kSortThreads + threadIdx.x;
        if (i < n) atomicAdd(&cnt[(keys[i] >> shift) & 0xFF], 1u);
    }
    __syncthreads();
    hist[(uint64_t)threadIdx.x * nb + blockIdx.x] = cnt[threadIdx.x];
}

// A block sorts its tile of 4,096 keys by the digit in LDS and writes it out in that order, so that the keys
// of a digit leave as one run (16 keys of a tile on average: a line) instead of one store a key.  A wave
// ranks its 1,024 keys in 16 rounds against counters of its own, so no round waits for another wave.  Bound
// by the memory: 16M keys 133 -> 67 us a pass for 270 MB read and written.
__global__ __launch_bounds__(kSortThreads) void k_radix_scatter(const uint64_t* __restrict__ in,
                                                                uint64_t* __restrict__ out, uint64_t n,
                                                                int shift,
                                                                const uint64_t* __restrict__ offsets,
                                                                uint32_t nb) {
    __shared__ uint64_t s_key[kSortTile];
    __shared__ uint32_t s_cnt[kSortWaves][256];   // a wave's keys per digit, then where they begin in the tile
    __shared__ uint64_t s_out[256];               // output index of the tile's first key, less its index here
    __shared__ uint32_t s_w[kSortWaves];
    const int t = threadIdx.x, wv = t >> 6, lane = t & 63;
    for (int w = 0; w < kSortWaves; ++w) s_cnt[w][t] = 0;
    __syncthreads();
    const uint64_t base = (uint64_t)blockIdx.x * kSortTile + (uint64_t)wv * (64 * kSortKeys) + lane;
    uint64_t key[kSortKeys];
    uint16_t rank[kSortKeys];
#pragma unroll
    for (int c = 0; c < kSortKeys; ++c) key[c] = base + c * 64 < n ? in[base + c * 64] : 0;
#pragma unroll
    for (int c = 0; c < kSortKeys; ++c) {
        const bool valid = base + c * 64 < n;
        const uint32_t d = (uint32_t)((key[c] >> shift) & 0xFF);
        uint64_t peers = __ballot(valid);
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            const bool bit = (d >> b) & 1;
            const uint64_t m = __ballot(bit);
            peers &= bit ? m : ~m;
        }
        const uint32_t before = s_cnt[wv][d];
        const uint32_t r = (uint32_t)__popcll(peers & rpqd::lanemask_lt());
        rank[c] = (uint16_t)(before + r);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        if (valid && r == 0) s_cnt[wv][d] = before + (uint32_t)__popcll(peers);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }
    __syncthreads();
    // thread t takes digit t: its keys over the waves, and their prefix over the digits
    uint32_t c[kSortWaves], sum = 0;
#pragma unroll
    for (int w = 0; w < kSortWaves; ++w) {
        c[w] = s_cnt[w][t];
        sum += c[w];
    }
    const uint32_t incl = rpqd::wave_incl_scan_u32(sum);
    if (lane == 63) s_w[wv] = incl;
    __syncthreads();
    uint32_t run = incl - sum;
    for (int w = 0; w < wv; ++w) run += s_w[w];
    s_out[t] = offsets[(uint64_t)t * nb + blockIdx.x] - run;
#pragma unroll
    for (int w = 0; w < kSortWaves; ++w) {
        s_cnt[w][t] = run;
        run += c[w];
    }
    __syncthreads();
#pragma unroll
    for (int c2 = 0; c2 < kSortKeys; ++c2)
        if (base + c2 * 64 < n) s_key[s_cnt[wv][(key[c2] >> shift) & 0xFF] + rank[c2]] = key[c2];
    __syncthreads();
    const uint32_t here = (uint32_t)min((uint64_t)kSortTile, n - (uint64_t)blockIdx.x * kSortTile);
    for (uint32_t i = t; i < here; i += kSortThreads) {
        const uint64_t k = s_key[i];
        out[s_out[(k >> shift) & 0xFF] + i] = k;
    }
}

uint64_t radix_temp_bytes(uint64_t n) {
    const uint64_t nb = (n + kSortTile - 1) / kSortTile;
    const uint64_t h = 256 * (nb ? nb : 1);
    return (h + scan_temp_elems(h) + 1) * sizeof(uint64_t);
}

int radix_sort_u64(uint64_t* keys, uint64_t* alt, uint64_t n, int lo_bits, int hi_bits, void* temp,
                   hipStream_t s, uint64_t** sorted) {
    *sorted = keys;
    if (n <= 1) return RPQ_OK;
    const uint64_t nb = (n + kSortTile - 1) / kSortTile;
    if (nb > 0xFFFFFFFFull) {
        set_error("radix sort input too large");
        return RPQ_EUNSUPPORTED;
    }
    uint64_t* hist = reinterpret_cast<uint64_t*>(temp);
    uint64_t* stemp = hist + 256 * nb;
    uint64_t* a = keys;
    uint64_t* b = alt;
    int shifts[16];
    int ns = 0;
    for (int sh = 0; sh < lo_bits && sh < 32; sh += 8) shifts[ns++] = sh;
    for (int sh = 32; sh < 32 + hi_bits && sh < 64; sh += 8) shifts[ns++] = sh;
    for (int i = 0; i < ns; ++i) {
        hipLaunchKernelGGL(k_radix_hist, dim3((unsigned)nb), dim3(kSortThreads), 0, s, a, n, shifts[i], hist,
                           (uint32_t)nb);
        RPQ_LAUNCH_CHECK();
        RPQ_TRY(exclusive_scan_u64(hist, hist, 256 * nb, stemp, nullptr, s));
        hipLaunchKernelGGL(k_radix_scatter, dim3((unsigned)nb), dim3(kSortThreads), 0, s, a, b, n, shifts[i],
                           hist, (uint32_t)nb);
        RPQ_LAUNCH_CHECK();
        uint64_t* t = a;
        a = b;
        b = t;
    }
    *sorted = a;
    return RPQ_OK;
}

}  // namespace rpq

namespace rpq {

uint64_t* host_stage() {
    thread_local uint64_t* stage = nullptr;
    if (!stage) {
        void* p = nullptr;
        if (hipHostMalloc(&p, 4096) == hipSuccess) stage = static_cast<uint64_t*>(p);
    }
    return stage;
}

}  // namespace rpq
