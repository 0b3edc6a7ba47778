// Sort of items by digits of their order-preserving keys.
//
// Without NaN every filter of the quicksort of Section 4 (Listing 3) keeps each item on one
// side of every pivot, and items that compare equal (-0 and +0 included) stay together in
// input order, so the listing's result is the stable sort of the input, whatever the pivots.
// A least-significant-digit radix sort computes that sort in at most four passes over the
// data where the recursion takes about 2 log2(n / 2048) levels.
//
// No filter keeps a NaN.  So the first pivot decides: if it is a NaN, the three filters are empty
// and so is the result; if not, every NaN is gone after the first level and the result is the
// stable sort of the others.  The passes then give NaN the largest key (which no number has), and
// the result ends before them.
//
// The items keep their bits (a -0 stays a -0); a pass extracts its 8-bit digit from the key:
// int32 by value, float32 by value with both zeros one key.  Keys are taken relative to the
// smallest one, so a range of fewer than 2^8, 2^16 or 2^24 keys needs one, two or three passes.
// A pass is three kernels.  The input is cut into chunks of whole tiles; r_hist counts each
// chunk's digits, r_scan turns the counts into offsets (one block per digit, over the chunks),
// and r_scatter walks its chunk tile by tile with a running offset per digit.  Nothing waits on
// another block.  (A single-pass scheme saves r_hist's read, 4 of 12 bytes per item and pass, and has
// its blocks poll each other's prefixes across the XCDs' L2s; not tried.)
//
// 10^8 float32 (four passes), with both postconditions: 1.57 ms; 13.9 ms by the recursion's
// levels.  Per pass r_hist 95-105 us (4 TB/s), r_scan 6 us, r_scatter 246 us (3.3 TB/s; 163 us
// would be a copy's).  200,003 int32 in [-25000, 25000] (two passes): 71 us, before 763 us.  One NaN
// among 10^8: 1.50 ms, before 14.5; among 3000: 72 us, before 313.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "sg_runtime.h"

namespace sgr {

constexpr int RB = 512;           // threads per block
constexpr int RW = RB / 64;       // waves per block
constexpr int RD = 256;           // digits
constexpr int RCOPY = 16;         // copies of a digit's counter in r_hist

struct KeyInfo {
    uint32_t min, max;  // of the keys
    uint32_t nan;       // items that are NaN
    uint32_t pivot;     // 1: the listing's first pivot is one
};

enum Kind { INT, FLT, NANS };  // int32, float32 without NaN, float32

__device__ __forceinline__ bool is_nan(uint32_t u) { return (u & 0x7FFFFFFFu) > 0x7F800000u; }

// Order-preserving unsigned key.  x + 0 maps -0 to +0 and leaves every other number as it is.
// (NaN keys take two instructions more per item, so only inputs with a NaN scatter by them.)
template <Kind F>
__device__ __forceinline__ uint32_t rkey(uint32_t u) {
    if (F == INT) return u ^ 0x80000000u;
    const bool nan = F == NANS && is_nan(u);
    u = __builtin_bit_cast(uint32_t, __builtin_bit_cast(float, u) + 0.0f);
    u ^= (uint32_t)(((int32_t)u >> 31) | (int32_t)0x80000000);
    return nan ? ~0u : u;
}

// Digit counts of one chunk (cnt[digit][chunk]); FIRST: also the keys' range and how many
// items are NaN.  Bound by the read.  A digit has 16 counters, one per lane modulo 16, so that
// equal digits (the exponent byte of ordinary floats has a handful of values) serialize at most
// four lanes of an LDS atomic.
template <Kind F, bool FIRST>
__global__ __launch_bounds__(RB) void r_hist(const uint32_t* __restrict__ a, int64_t n, int64_t chunk, uint32_t bias,
                                             int shift, uint32_t* __restrict__ cnt, KeyInfo* __restrict__ info) {
    __shared__ uint32_t h[RD * RCOPY];
    __shared__ uint32_t smin[RW], smax[RW], snan[RW];
    const int tid = threadIdx.x;
    for (int i = tid; i < RD * RCOPY; i += RB) h[i] = 0;
    __syncthreads();
    const int64_t lo = (int64_t)blockIdx.x * chunk, hi = std::min<int64_t>(lo + chunk, n);
    const int c = tid & (RCOPY - 1);
    if (FIRST && F != INT && tid == 0 && n / 2 >= lo && n / 2 < hi && is_nan(a[n / 2])) info->pivot = 1u;
    uint32_t kmin = ~0u, kmax = 0u, nan = 0u;
    auto take = [&](uint32_t u) {
        const uint32_t k = rkey<F>(u);
        if (FIRST) {
            kmin = min(kmin, k);
            kmax = max(kmax, k);
            if (F != INT) nan += is_nan(u) ? 1u : 0u;
        }
        atomicAdd(&h[(((k - bias) >> shift) & (RD - 1)) * RCOPY + c], 1u);
    };
    constexpr int Q = 4;  // 16-byte loads in flight per thread
    int64_t i = lo;
    if ((reinterpret_cast<uintptr_t>(a) & 15) == 0) {  // chunks start at multiples of a tile
        for (; i + RB * 4 * Q <= hi; i += RB * 4 * Q) {
            uint4 x[Q];
#pragma unroll
            for (int q = 0; q < Q; ++q) x[q] = *reinterpret_cast<const uint4*>(a + i + (q * RB + tid) * 4);
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                take(x[q].x);
                take(x[q].y);
                take(x[q].z);
                take(x[q].w);
            }
        }
    }
    for (; i < hi; i += RB * Q) {
        uint32_t x[Q];
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const int64_t j = i + q * RB + tid;
            x[q] = j < hi ? a[j] : 0u;
        }
#pragma unroll
        for (int q = 0; q < Q; ++q)
            if (i + q * RB + tid < hi) take(x[q]);
    }
    if (FIRST) {
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            kmin = min(kmin, (uint32_t)__shfl_xor(kmin, o));
            kmax = max(kmax, (uint32_t)__shfl_xor(kmax, o));
            nan += __shfl_xor(nan, o);
        }
        if ((tid & 63) == 0) {
            smin[tid >> 6] = kmin;
            smax[tid >> 6] = kmax;
            snan[tid >> 6] = nan;
        }
    }
    __syncthreads();
    if (tid < RD) {
        uint32_t s = 0;
#pragma unroll
        for (int k = 0; k < RCOPY; ++k) s += h[tid * RCOPY + ((tid + k) & (RCOPY - 1))];
        cnt[(int64_t)tid * gridDim.x + blockIdx.x] = s;
    }
    if (FIRST && tid == 0) {
        for (int w = 1; w < RW; ++w) {
            kmin = min(kmin, smin[w]);
            kmax = max(kmax, smax[w]);
            nan += snan[w];
        }
        atomicMin(&info->min, kmin);
        atomicMax(&info->max, kmax);
        if (nan) atomicAdd(&info->nan, nan);
    }
}

__device__ __forceinline__ uint32_t wave_incl(uint32_t v, int lane) {
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t y = __shfl_up(v, o);
        if (lane >= o) v += y;
    }
    return v;
}

// One block per digit: its chunk counts become exclusive offsets; tot[digit] their sum.
__global__ __launch_bounds__(256) void r_scan(uint32_t* __restrict__ cnt, uint32_t* __restrict__ tot, int chunks) {
    __shared__ uint32_t ws[4];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    uint32_t* row = cnt + (int64_t)blockIdx.x * chunks;
    uint32_t carry = 0;
    for (int c0 = 0; c0 < chunks; c0 += 256) {
        const uint32_t v = c0 + tid < chunks ? row[c0 + tid] : 0u;
        const uint32_t incl = wave_incl(v, lane);
        if (lane == 63) ws[wave] = incl;
        __syncthreads();
        uint32_t base = carry, all = 0;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            if (w < wave) base += ws[w];
            all += ws[w];
        }
        if (c0 + tid < chunks) row[c0 + tid] = base + incl - v;
        carry += all;
        __syncthreads();
    }
    if (tid == 0) tot[blockIdx.x] = carry;
}

// Move one chunk's items to their places for this digit.  A wave holds I rows of 64
// consecutive items of the tile; a row's items of equal digit find each other by eight ballots
// (one per digit bit), so an item's rank is its wave's count of the digit so far plus the lanes
// below it: no lane-order assumption on LDS atomics, and stable.  The tile is then staged in
// LDS in digit order, so that a digit's items leave as one contiguous run.  Registers are held
// to 128 for two workgroups per CU: each hides the other's barriers and rank chains (10^8
// float32: 411 us a pass with 133 registers and one workgroup, 320 with two; three, at 80
// registers with spills, 420).  Vector instructions fill two thirds of it, so the ballots' part
// is kept to four a bit (bit, comparison, two three-input logic operations), whole tiles have no
// conditions, and LDS reads go in batches: 296 -> 246 us.  Finding equal digits by atomic ORs of
// lane masks in LDS is no faster on spread digits and half as fast on equal ones; loading the
// next tile ahead spills.
template <Kind F, int I>
__global__ __launch_bounds__(RB, I == 4 ? 2 : 4) void r_scatter(const uint32_t* __restrict__ a, uint32_t* __restrict__ out,
                                                               int64_t n, int64_t chunk, uint32_t bias, int shift,
                                                               const uint32_t* __restrict__ cnt,
                                                               const uint32_t* __restrict__ tot) {
    constexpr int TILE = RB * I;
    __shared__ uint32_t stage[TILE];
    __shared__ uint32_t wh[RW][RD];   // per wave: counts, then first place in the staged tile
    __shared__ uint32_t goff[RD];     // where the digit's next item goes, less its staged place
    __shared__ uint32_t ws[RD / 64];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    // exclusive prefix over the digits (all threads run it; the first RD hold one digit each)
    auto digit_excl = [&](uint32_t v) -> uint32_t {
        const uint32_t incl = wave_incl(v, lane);
        if (lane == 63 && wave < RD / 64) ws[wave] = incl;
        __syncthreads();
        uint32_t base = 0;
#pragma unroll
        for (int w = 0; w < RD / 64; ++w)
            if (w < wave) base += ws[w];
        return base + incl - v;
    };
    uint32_t gnext = digit_excl(tid < RD ? tot[tid] : 0u);  // of digit tid, kept by its thread
    if (tid < RD) gnext += cnt[(int64_t)tid * gridDim.x + blockIdx.x];
    const int64_t lo = (int64_t)blockIdx.x * chunk, hi = std::min<int64_t>(lo + chunk, n);
    const int first = wave * 64 * I + lane;
    auto tile = [&](auto full, int64_t t0) {
        constexpr bool FULL = decltype(full)::value;
        const int m = FULL ? TILE : (int)(hi - t0);
        uint32_t x[I];
        // read once: left out of the L2's lines, which collect the runs being written
        if (FULL) {
#pragma unroll
            for (int i = 0; i < I; ++i) x[i] = __builtin_nontemporal_load(a + t0 + first + 64 * i);
        } else {
#pragma unroll
            for (int i = 0; i < I; ++i) x[i] = first + 64 * i < m ? a[t0 + first + 64 * i] : 0u;
        }
        for (int i = tid; i < RW * RD; i += RB) (&wh[0][0])[i] = 0;
        __syncthreads();
        // rank | digit << 16: places past the end take the last digit, so they are staged last
        uint32_t rd[I];
#pragma unroll
        for (int i = 0; i < I; ++i) {
            uint32_t d = ((rkey<F>(x[i]) - bias) >> shift) & (RD - 1);
            if (!FULL && first + 64 * i >= m) d = RD - 1;
            uint32_t mlo = ~0u, mhi = ~0u;
            int32_t sb[8];
            uint64_t bal[8];
#pragma unroll
            for (int b = 0; b < 8; ++b) {
                sb[b] = __builtin_amdgcn_sbfe((int)d, b, 1);
                asm("" : "+v"(sb[b]));  // else the comparison gets a shift of its own
                bal[b] = __ballot(sb[b] != 0);
            }
            // m & ~(ballot ^ s) in one operation
#pragma unroll
            for (int b = 0; b < 8; ++b) {
                mlo = __builtin_amdgcn_bitop3_b32(mlo, (uint32_t)bal[b], (uint32_t)sb[b], 0x90);
                mhi = __builtin_amdgcn_bitop3_b32(mhi, (uint32_t)(bal[b] >> 32), (uint32_t)sb[b], 0x90);
            }
            const uint32_t below = __builtin_amdgcn_mbcnt_hi(mhi, __builtin_amdgcn_mbcnt_lo(mlo, 0u));
            // the wave's LDS accesses keep their order: every lane of the row reads the count
            // before the group's first lane advances it (an add: nothing waits for the read)
            const uint32_t prev = __hip_atomic_load(&wh[wave][d], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            __builtin_amdgcn_wave_barrier();
            if (below == 0)
                __hip_atomic_fetch_add(&wh[wave][d], (uint32_t)(__builtin_popcount(mlo) + __builtin_popcount(mhi)),
                                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            __builtin_amdgcn_wave_barrier();
            rd[i] = (prev + below) | (d << 16);
        }
        __syncthreads();
        uint32_t mine = 0;
        uint32_t wc[RW];
        if (tid < RD) {
#pragma unroll
            for (int w = 0; w < RW; ++w) {
                wc[w] = mine;
                mine += wh[w][tid];
            }
        }
        const uint32_t place = digit_excl(mine);  // first staged place of digit tid
        if (tid < RD) {
#pragma unroll
            for (int w = 0; w < RW; ++w) wh[w][tid] = place + wc[w];
            goff[tid] = gnext - place;
            gnext += mine;
        }
        __syncthreads();
        uint32_t q[I];
#pragma unroll
        for (int i = 0; i < I; ++i) q[i] = wh[wave][rd[i] >> 16];
#pragma unroll
        for (int i = 0; i < I; ++i) stage[q[i] + (rd[i] & 0xFFFFu)] = x[i];
        __syncthreads();
        constexpr int G = I < 8 ? I : 8;  // LDS reads in flight
#pragma unroll
        for (int i0 = 0; i0 < I; i0 += G) {
            uint32_t v[G], g[G];
#pragma unroll
            for (int i = 0; i < G; ++i) v[i] = stage[tid + RB * (i0 + i)];
#pragma unroll
            for (int i = 0; i < G; ++i) g[i] = goff[((rkey<F>(v[i]) - bias) >> shift) & (RD - 1)];
#pragma unroll
            for (int i = 0; i < G; ++i) {
                const int p = tid + RB * (i0 + i);
                if (FULL || p < m) out[g[i] + (uint32_t)p] = v[i];
            }
        }
        // the next tile's counters and staging overwrite what this one reads only after its
        // own first barriers: wh after the barrier above, goff and stage after two more
    };
    for (int64_t t0 = lo; t0 < hi; t0 += TILE) {
        if (t0 + TILE <= hi) tile(std::true_type{}, t0);
        else tile(std::false_type{}, t0);
    }
}

__global__ void r_info_init(KeyInfo* info) { *info = KeyInfo{~0u, 0u, 0u, 0u}; }

}  // namespace sgr

namespace sgrt {

// The quicksort of m items (2 <= m < 2^32) from src to dst; *count of them are in the result.
sg_status radix_sort(sg_ctx_s* ctx, const uint32_t* src, uint32_t* dst, int64_t m, bool is_f32, int64_t* count) {
    using namespace sgr;
    hipStream_t st = ctx->stream;
    const bool small = m < (int64_t)ctx->num_cu * RB * 16;
    const int64_t tile = small ? RB * 4 : RB * 16;
    const int64_t tiles = (m + tile - 1) / tile;
    const int64_t per = (tiles + (int64_t)ctx->num_cu * 6 - 1) / ((int64_t)ctx->num_cu * 6);
    const int64_t chunk = per * tile;
    const int chunks = (int)((m + chunk - 1) / chunk);
    auto up = [](size_t b) { return (b + 255) & ~(size_t)255; };
    const size_t b_items = up((size_t)m * 4), b_cnt = up((size_t)RD * chunks * 4), b_tot = up(RD * 4);
    char* w = (char*)dev_alloc(ctx, b_items + b_cnt + b_tot + 256);
    if (!w) return fail(ctx, SG_E_OOM, "quicksort: work memory");
    uint32_t* tmp = (uint32_t*)w;
    uint32_t* cnt = (uint32_t*)(w + b_items);
    uint32_t* tot = (uint32_t*)(w + b_items + b_cnt);
    KeyInfo* info = (KeyInfo*)(w + b_items + b_cnt + b_tot);
    KeyInfo h{};
    hipError_t e = hipSuccess;
    const dim3 g((unsigned)chunks), b(RB);
#define SGR_HIST(F, FIRST) hipLaunchKernelGGL((r_hist<F, FIRST>), g, b, 0, st, from, m, chunk, bias, shift, cnt, info)
#define SGR_SCATTER(F, I) hipLaunchKernelGGL((r_scatter<F, I>), g, b, 0, st, from, to, m, chunk, bias, shift, cnt, tot)
    auto first_hist = [&](const uint32_t* from, uint32_t bias, int shift) {
        if (is_f32) SGR_HIST(NANS, true);
        else SGR_HIST(INT, true);
    };
    // the first count is taken before the keys' range is known; the range's lower end is cut to
    // a multiple of 256, so the lowest digit is the same with and without it
    hipLaunchKernelGGL(r_info_init, dim3(1), dim3(1), 0, st, info);
    first_hist(src, 0u, 0);
    if (e == hipSuccess) e = hipGetLastError();
    if (e == hipSuccess) e = hipMemcpyAsync(&h, info, sizeof(h), hipMemcpyDeviceToHost, st);
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    if (e != hipSuccess || h.pivot) {
        dev_free(ctx, w);
        *count = 0;
        return e != hipSuccess ? hip_fail(ctx, e, "quicksort: digit count") : SG_OK;
    }
    const Kind kind = !is_f32 ? INT : h.nan ? NANS : FLT;
    const uint32_t bias = h.min & ~(uint32_t)(RD - 1), range = h.max - bias;
    int passes = 1;
    while (passes < 4 && (range >> (8 * passes)) != 0) ++passes;
    const uint32_t* from = src;
    for (int p = 0; p < passes && e == hipSuccess; ++p) {
        uint32_t* to = (passes - 1 - p) % 2 == 0 ? dst : tmp;
        const int shift = 8 * p;
        if (p > 0) {
            if (kind == INT) SGR_HIST(INT, false);
            else if (kind == FLT) SGR_HIST(FLT, false);
            else SGR_HIST(NANS, false);
        }
        hipLaunchKernelGGL(r_scan, dim3(RD), dim3(256), 0, st, cnt, tot, chunks);
        if (small) {
            if (kind == INT) SGR_SCATTER(INT, 4);
            else if (kind == FLT) SGR_SCATTER(FLT, 4);
            else SGR_SCATTER(NANS, 4);
        } else {
            if (kind == INT) SGR_SCATTER(INT, 16);
            else if (kind == FLT) SGR_SCATTER(FLT, 16);
            else SGR_SCATTER(NANS, 16);
        }
        e = hipGetLastError();
        from = to;
    }
#undef SGR_SCATTER
#undef SGR_HIST
    // the pool hands the block out again in stream order only
    dev_free(ctx, w);
    if (e != hipSuccess) return hip_fail(ctx, e, "quicksort: digit pass");
    *count = m - h.nan;
    return SG_OK;
}

}  // namespace sgrt
