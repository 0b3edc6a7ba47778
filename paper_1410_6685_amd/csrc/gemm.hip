// Matrix product C = A B on the FP32 matrix cores (Section 3.4: the matrix class multiplies
// row-major matrices using on-chip shared memory).
//
// v_mfma_f32_32x32x2f32: each wave multiplies a 32x2 by a 2x32 block per instruction and
// accumulates a 32x32 fp32 tile.  A 256-thread block computes a T x T tile of C (T = 128: each
// wave 64x64 = 2x2 MFMA tiles; T = 64: one), streaming K slices of A and B through LDS;
// registers hold the next slice while the current one is consumed.  Blocks are reordered so
// that the tiles of C one XCD holds at a time form a square patch whose panels its L2 shares.
//
// Matrices too small to give every CU a 128 x 128 tile run on 64 x 64 ones, and if those are
// fewer than two per CU, K is cut into parts whose products are added in order by a second
// kernel (the sums' rounding errors shrink with it).  Before (128 x 128 tiles only, guarded
// loads on unaligned rows) and now: 1000 x 1531 x 777 181 and 44 us, 1024^3 85 and 34 us,
// 64 x 4096 x 64 497 and 20 us, 4095 x 4095 x 4093 1583 and 1005 us, 4096^3 1067 and 1005 us
// (137 TFLOP/s of the matrix cores' 157 in FP32, which are busy 87 % of the cycles).
//
// The bfloat16 cores, on three parts per value, are no way round that bound.  With six of the
// nine part products 4096^3 takes 706 us (986 here, alone), but a single product is off by up to 1.4 units in the
// last place (here 0.5; a diagonal or selecting factor shows it).  Eight, the small ones added up
// apart, bring that to 0.51 and halve a dense sum's error, and then 2048^3 takes 161 us against
// 159 here; a 256-wide tile no longer fits the registers.
//
// Operands are read through buffer descriptors of the block's rows: a row past the matrix is out of the buffer's
// range and reads as zero, so no lane branches around a load (a divergent branch makes the
// compiler wait for every load in flight), and 16-byte loads need no more than the 4-byte
// alignment that every matrix has.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

namespace sg {

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

constexpr int APAD = 1, BPAD = 4;

__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc(const float* p, int64_t elems) {
    const uint32_t bytes = elems >= (1 << 30) ? 0xFFFFFFFFu : (uint32_t)(elems * 4);
    return __builtin_amdgcn_make_buffer_rsrc((void*)p, 0, (int)bytes, 0x00020000);
}

// Offsets within a tile's rows of A (T * K floats) and a slice's rows of B fit 32 bits.
constexpr int64_t GBUF_MAX_K = 1 << 23, GBUF_MAX_N = 1 << 24;

// T: tile of C (64 or 128); GBK: depth of a K slice; NBUF: LDS buffers (2: the next slice is
// stored while the current one is consumed, one barrier per slice; 1: two barriers per slice,
// half the LDS); BIG: rows longer than 32-bit offsets reach, loaded element by element.  Part z
// of the K range, [z * kpart, (z + 1) * kpart), goes to C + z * M * N.
template <int T, int GBK, int NBUF, bool BIG = false>
__global__ __launch_bounds__(256) void gemm_f32_kernel(const float* __restrict__ A, const float* __restrict__ B,
                                                       float* __restrict__ C, int M, int N, int K, int kpart) {
    constexpr int W = T / 64;       // MFMA tiles of a wave along each side
    constexpr int AQ = GBK / 4;     // 16-byte loads per row of an A slice
    constexpr int BQ = T / 4;       // and of a B slice
    constexpr int P = T * AQ / 256; // of each per thread
    static_assert(T * AQ % 256 == 0, "slice");
    __shared__ float As[NBUF][T][GBK + APAD];
    __shared__ float Bs[NBUF][GBK][T + BPAD];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int tiles_m = (M + T - 1) / T, tiles_n = (N + T - 1) / T;
    const int nb = gridDim.x;
    int tile = blockIdx.x;
    if ((nb & 7) == 0) tile = (blockIdx.x & 7) * (nb >> 3) + (blockIdx.x >> 3);  // XCD-contiguous
    // tiles in groups of 8 tile rows, column by column within a group: the blocks resident on
    // one XCD at a time cover an 8 x 8 patch of C, so they share 8 slices of A and 8 of B
    // (a row-major order would need 2 of A and 32 of B)
    constexpr int G = 8;
    const int width = G * tiles_n;
    const int first = (tile / width) * G;
    const int gs = tiles_m - first < G ? tiles_m - first : G;
    const int m0 = (first + (tile % width) % gs) * T, n0 = ((tile % width) / gs) * T;
    const int wm = (wave >> 1) * (T / 2), wn = (wave & 1) * (T / 2);
    const int kb = (int)blockIdx.y * kpart, ke = kb + kpart < K ? kb + kpart : K;
    const auto ra = rsrc(A + (int64_t)m0 * K, (int64_t)(M - m0) * K);

    floatx16 acc[W][W];
#pragma unroll
    for (int i = 0; i < W; ++i)
#pragma unroll
        for (int j = 0; j < W; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

    u32x4 va[P], vb[P];
    auto load = [&](int k0) {
        if (BIG) {
#pragma unroll
            for (int p = 0; p < P; ++p) {
                const int idx = tid + 256 * p;
                const int gm = m0 + idx / AQ, kq = k0 + (idx % AQ) * 4, kr = k0 + idx / BQ, gn = n0 + (idx % BQ) * 4;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    va[p][q] = gm < M && kq + q < ke ? __builtin_bit_cast(uint32_t, A[(int64_t)gm * K + kq + q]) : 0u;
                    vb[p][q] = kr < ke && gn + q < N ? __builtin_bit_cast(uint32_t, B[(int64_t)kr * N + gn + q]) : 0u;
                }
            }
            return;
        }
        const auto rb = rsrc(B + (int64_t)k0 * N, (int64_t)(K - k0) * N);
        const uint32_t ka = (uint32_t)k0 * 4;
        if (k0 + GBK <= ke && k0 + GBK + (N == 1 ? 3 : 1) <= K) {
            // whole slice: a row of A past M starts past the buffer's end, and what follows a
            // row's end (columns of B past N) feeds columns of C that are not stored.  16 bytes that
            // hold a stored column end at most three values into the row behind (one column: into
            // the three rows behind), which exists, so those that straddle the buffer's end hold
            // nothing that is stored
#pragma unroll
            for (int p = 0; p < P; ++p) {
                const uint32_t idx = tid + 256 * p;
                va[p] = __builtin_amdgcn_raw_buffer_load_b128(ra, ((idx / AQ) * (uint32_t)K + (idx % AQ) * 4) * 4 + ka, 0, 0);
                vb[p] = __builtin_amdgcn_raw_buffer_load_b128(rb, ((idx / BQ) * (uint32_t)N + (uint32_t)n0 + (idx % BQ) * 4) * 4, 0, 0);
            }
            return;
        }
        // the last slice: element by element, k past the part's end as zero in A and in B
#pragma unroll
        for (int p = 0; p < P; ++p) {
            const uint32_t idx = tid + 256 * p;
            const uint32_t ia = (idx % AQ) * 4, ib = idx / BQ;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const uint32_t x = __builtin_amdgcn_raw_buffer_load_b32(ra, ((idx / AQ) * (uint32_t)K + ia + q) * 4 + ka, 0, 0);
                va[p][q] = k0 + (int)ia + q < ke ? x : 0u;
                const uint32_t y = __builtin_amdgcn_raw_buffer_load_b32(rb, (ib * (uint32_t)N + (uint32_t)n0 + (idx % BQ) * 4 + q) * 4, 0, 0);
                vb[p][q] = k0 + (int)ib < ke ? y : 0u;
            }
        }
    };
    auto store = [&](int buf) {
#pragma unroll
        for (int p = 0; p < P; ++p) {
            const int idx = tid + 256 * p;
#pragma unroll
            for (int q = 0; q < 4; ++q) As[buf][idx / AQ][(idx % AQ) * 4 + q] = __builtin_bit_cast(float, (uint32_t)va[p][q]);
#pragma unroll
            for (int q = 0; q < 4; ++q) Bs[buf][idx / BQ][(idx % BQ) * 4 + q] = __builtin_bit_cast(float, (uint32_t)vb[p][q]);
        }
    };

    const int nk = (ke - kb + GBK - 1) / GBK;
    load(kb);
    store(0);
    __syncthreads();
    const int li = lane & 31, lk = lane >> 5;
    for (int kt = 0; kt < nk; ++kt) {
        const int buf = NBUF == 2 ? (kt & 1) : 0;
        if (kt + 1 < nk) load(kb + (kt + 1) * GBK);
#pragma unroll
        for (int kk = 0; kk < GBK; kk += 2) {
            float a[W], b[W];
#pragma unroll
            for (int t = 0; t < W; ++t) {
                a[t] = As[buf][wm + 32 * t + li][kk + lk];
                b[t] = Bs[buf][kk + lk][wn + 32 * t + li];
            }
#pragma unroll
            for (int i = 0; i < W; ++i)
#pragma unroll
                for (int j = 0; j < W; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i], b[j], acc[i][j], 0, 0, 0);
        }
        if (NBUF == 1) __syncthreads();  // every wave is done with the buffer
        if (kt + 1 < nk) store(NBUF == 2 ? (buf ^ 1) : 0);
        __syncthreads();
    }
    // accumulator layout: register r of lane l holds row 8*(r/4) + 4*(l/32) + (r%4), column l%32
    float* out = C + (int64_t)blockIdx.y * M * N;
#pragma unroll
    for (int i = 0; i < W; ++i)
#pragma unroll
        for (int j = 0; j < W; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int row = m0 + wm + 32 * i + 8 * (r >> 2) + 4 * lk + (r & 3);
                const int col = n0 + wn + 32 * j + li;
                if (row < M && col < N) out[(int64_t)row * N + col] = acc[i][j][r];
            }
}

// C = the sum of the K parts' products, in order.
__global__ __launch_bounds__(256) void gemm_sum_kernel(const float* __restrict__ part, float* __restrict__ C, int64_t mn,
                                                       int parts) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= mn) return;
    float s = part[i];
    for (int z = 1; z < parts; ++z) s += part[z * mn + i];
    C[i] = s;
}

}  // namespace sg

// Parts of K the product is computed in (1: no work memory needed).
int sg_gemm_parts(int64_t M, int64_t N, int64_t K, int num_cu) {
    const int64_t t128 = ((M + 127) / 128) * ((N + 127) / 128), t64 = ((M + 63) / 64) * ((N + 63) / 64);
    if (K > sg::GBUF_MAX_K || N > sg::GBUF_MAX_N || t128 >= num_cu) return 1;
    // two blocks per CU; a part is at least 128 deep, so that adding the parts stays small beside it
    return (int)std::max<int64_t>(1, std::min<int64_t>((int64_t)num_cu * 2 / t64, K / 128));
}

// work: sg_gemm_parts() * M * N floats when that is more than one part; without it K stays in one.
hipError_t sg_launch_gemm_f32(const float* A, const float* B, float* C, int64_t M, int64_t N, int64_t K, int num_cu,
                              float* work, hipStream_t s) {
    if (M <= 0 || N <= 0) return hipSuccess;
    if (M > (1 << 30) || N > (1 << 30) || K > (1 << 30)) return hipErrorInvalidValue;
    const int64_t t128 = ((M + 127) / 128) * ((N + 127) / 128), t64 = ((M + 63) / 64) * ((N + 63) / 64);
    if (t64 > (1 << 30)) return hipErrorInvalidValue;
    const int parts = work ? sg_gemm_parts(M, N, K, num_cu) : 1;
    float* out = parts > 1 ? work : C;
    int64_t kpart = (K + parts - 1) / parts;
    kpart = std::max<int64_t>(1, parts > 1 ? (kpart + 31) / 32 * 32 : K);
    if (K > sg::GBUF_MAX_K || N > sg::GBUF_MAX_N)
        hipLaunchKernelGGL((sg::gemm_f32_kernel<128, 16, 1, true>), dim3((unsigned)t128), dim3(256), 0, s, A, B, out, (int)M,
                           (int)N, (int)K, (int)kpart);
    else if (t128 >= num_cu)
        hipLaunchKernelGGL((sg::gemm_f32_kernel<128, 16, 1>), dim3((unsigned)t128), dim3(256), 0, s, A, B, out, (int)M, (int)N,
                           (int)K, (int)kpart);
    else
        hipLaunchKernelGGL((sg::gemm_f32_kernel<64, 32, 2>), dim3((unsigned)t64, (unsigned)std::max<int64_t>(1, (K + kpart - 1) / kpart)), dim3(256),
                           0, s, A, B, out, (int)M, (int)N, (int)K, (int)kpart);
    if (parts > 1)
        hipLaunchKernelGGL(sg::gemm_sum_kernel, dim3((unsigned)((M * N + 255) / 256)), dim3(256), 0, s, (const float*)work, C, M * N,
                           (int)((K + kpart - 1) / kpart));
    return hipGetLastError();
}
