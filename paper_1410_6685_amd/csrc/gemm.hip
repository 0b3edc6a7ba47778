// Matrix product C = A B on the FP32 matrix cores (Section 3.4: the matrix class multiplies
// row-major matrices using on-chip shared memory).
//
// v_mfma_f32_32x32x2f32: each wave multiplies a 32x2 by a 2x32 block per instruction and
// accumulates a 32x32 fp32 tile.  A 256-thread block computes a T x T tile of C (T = 128: each
// wave 64x64 = 2x2 MFMA tiles; T = 64: one), streaming K slices of A and B through LDS;
// registers hold the next slice while the current one is consumed.  Blocks are reordered so
// that the tiles of C one XCD holds at a time form a square patch whose panels its L2 shares.
//
// Large products run on the bfloat16 matrix cores, on three parts per value (below).
//
// Matrices too small to give every CU a 128 x 128 tile run on 64 x 64 ones, and if those are
// fewer than two per CU, K is cut into parts whose products are added in order by a second
// kernel (the sums' rounding errors shrink with it).  Before (128 x 128 tiles only, guarded
// loads on unaligned rows) and now: 1000 x 1531 x 777 181 and 45 us, 1024^3 87 and 34 us,
// 64 x 4096 x 64 497 and 18 us, 4095 x 4095 x 4093 1629 and 1147 us, 4096^3 1200 and 1140 us
// (120 TFLOP/s of the matrix cores' 157 in FP32; where a value has no parts).
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
                                                       float* __restrict__ C, int M, int N, int K, int kpart,
                                                       const uint32_t* __restrict__ only_if) {
    if (only_if && *only_if == 0) return;  // the product is computed another way
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

// ---- large products: three bfloat16 parts per value ------------------------------------------
//
// A float32 value is the exact sum of three bfloat16 ones, x = h + m + l, each the rounding of
// what is left (8 bits of the 24; |m| <= 2^-9 |x| and |l| <= 2^-18 |x|).  Of the nine products of
// parts, six are formed on the bfloat16 matrix cores (16 times the FP32 rate) and accumulated in
// float32: hh, hm, mh, mm, hl, lh.  The other three are below 2^-26 of the product, a quarter of
// a float32 rounding.  Exact wherever the float32 product is (a value times a power of two is
// h + m + l times one part).  Error against float64 (relative 2-norm), on the FP32 matrix cores
// and here: normal and uniform entries K = 512 4.1e-7 and 3.4e-7, K = 4096 1.15e-6 and 1.00e-6;
// positive entries K = 4096 8.4e-7 and 5.3e-7; magnitudes spread over 2^24 K = 4096 8.0e-7 and
// 7.1e-7: an MFMA adds 16 products between two float32 roundings, the FP32 one two.
// 4096^3: 690 us for 6 * 137 GFLOP (1.2 PFLOP/s; 500 us on zeros, the clock falls with the data's
// switching) and 65 us for the parts, before 1140 us.
//
// Parts must not leave bfloat16's normal range, nor their products float32's: a nonzero value
// below 2^-40 or a value of 2^60 or more (infinities and NaN among them) sets a flag, and the
// FP32 kernel runs instead (both are launched; one returns at once).

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
constexpr int SK = 16;  // depth of a slice: one MFMA

__device__ __forceinline__ uint32_t bf16_rn(float x) {  // finite x
    const uint32_t u = __builtin_bit_cast(uint32_t, x);
    return (u + 0x7FFFu + ((u >> 16) & 1u)) >> 16;
}

// The three parts of a matrix, laid out as the product reads them: slice by slice of 16 along K,
// per slice the T rows of a tile (columns, for B) in blocks of 32, each block's 1 KiB in the
// order of an MFMA operand (lane l: row l % 32, k = 8 (l / 32) .. + 7).  Past the matrix: zeros.
// One wave per 32 rows and two slices.
__global__ void gemm_flag_kernel(uint32_t* flag) { *flag = 0u; }

template <int T, bool IS_B>
__global__ __launch_bounds__(256) void gemm_split_kernel(const float* __restrict__ X, u32x4* __restrict__ P, int rows, int K,
                                                         int64_t ld, int KS, uint32_t* __restrict__ flag) {
    constexpr int RB = T / 32;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int rb = blockIdx.y;  // block of 32 rows
    const int r = rb * 32 + (lane & 31);
    bool odd = false;
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        const int ks = ((int)blockIdx.x * 4 + wave) * 2 + s;
        if (ks >= KS) break;
        const int k0 = ks * SK + (lane >> 5) * 8;
        uint32_t p[3][8];
        float x[8];
        if (!IS_B && r < rows && k0 + 8 <= K) {  // along a row: two 16-byte loads, at any alignment
            typedef float f4 __attribute__((ext_vector_type(4), aligned(4)));
            const f4 lo = *reinterpret_cast<const f4*>(X + (int64_t)r * ld + k0);
            const f4 hi = *reinterpret_cast<const f4*>(X + (int64_t)r * ld + k0 + 4);
#pragma unroll
            for (int i = 0; i < 4; ++i) { x[i] = lo[i]; x[4 + i] = hi[i]; }
        } else {
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const bool in = r < rows && k0 + i < K;
                x[i] = in ? (IS_B ? X[(int64_t)(k0 + i) * ld + r] : X[(int64_t)r * ld + k0 + i]) : 0.f;
            }
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const float a = __builtin_fabsf(x[i]);
            odd |= !(a < 0x1p60f) || (a < 0x1p-40f && a != 0.f);
            float v = x[i];
#pragma unroll
            for (int q = 0; q < 3; ++q) {
                p[q][i] = bf16_rn(v);
                v -= __builtin_bit_cast(float, p[q][i] << 16);  // exact
            }
        }
        u32x4* dst = P + ((((int64_t)(rb / RB) * KS + ks) * 3) * RB + rb % RB) * 64 + lane;
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            u32x4 w;
#pragma unroll
            for (int i = 0; i < 4; ++i) w[i] = p[q][2 * i] | (p[q][2 * i + 1] << 16);
            dst[(int64_t)q * RB * 64] = w;
        }
    }
    if (__ballot(odd) && lane == 0) *flag = 1u;
}

// A block of NW waves computes a T x T tile, a wave WM x WN MFMA tiles of 32 x 32 (eight waves:
// two per SIMD cover each other's LDS reads; four waves of 4 x 4 tiles took the same time at
// T = 256, 10% more at T = 128).  A slice's parts (T = 256: 48 KiB) are copied to LDS as they lie
// in memory, one buffer being filled from registers while the other is consumed.
template <int T, int NW>
__global__ __launch_bounds__(64 * NW, 1) void gemm_parts_kernel(const u32x4* __restrict__ PA, const u32x4* __restrict__ PB,
                                                            float* __restrict__ C, int M, int N, int KS,
                                                            const uint32_t* __restrict__ flag) {
    constexpr int RB = T / 32;
    constexpr int WC = NW / 2, WM = RB / 2, WN = RB / WC;  // waves 2 x WC, MFMA tiles of one WM x WN
    constexpr int CH = 3 * RB;        // KiB of a slice of A or B
    constexpr int Q = 2 * CH / NW;     // KiB copied by a wave
    __shared__ u32x4 smem[2][2 * CH * 64];
    if (*flag) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int tiles_m = (M + T - 1) / T, tiles_n = (N + T - 1) / T;
    const int nb = gridDim.x;
    int tile = blockIdx.x;
    if ((nb & 7) == 0) tile = (blockIdx.x & 7) * (nb >> 3) + (blockIdx.x >> 3);  // XCD-contiguous
    constexpr int G = 4;
    const int width = G * tiles_n;
    const int first = (tile / width) * G;
    const int gs = tiles_m - first < G ? tiles_m - first : G;
    const int tm = first + (tile % width) % gs, tn = (tile % width) / gs;
    const u32x4* pa = PA + (int64_t)tm * KS * CH * 64;
    const u32x4* pb = PB + (int64_t)tn * KS * CH * 64;

    floatx16 acc[WM][WN];
#pragma unroll
    for (int i = 0; i < WM; ++i)
#pragma unroll
        for (int j = 0; j < WN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

    u32x4 v[Q];
    auto load = [&](int ks) {
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const int c = wave * Q + q;  // the first half of the waves copies A, the second B
            v[q] = wave < NW / 2 ? pa[((int64_t)ks * CH + c) * 64 + lane] : pb[((int64_t)ks * CH + c - CH) * 64 + lane];
        }
    };
    auto store = [&](int buf) {
#pragma unroll
        for (int q = 0; q < Q; ++q) smem[buf][(wave * Q + q) * 64 + lane] = v[q];
    };
    load(0);
    store(0);
    __syncthreads();
    const int am = wave / WC * WM, bn = wave % WC * WN;  // first block of 32 rows / columns
    for (int ks = 0; ks < KS; ++ks) {
        const u32x4* sa = smem[ks & 1];
        const u32x4* sb = sa + CH * 64;
        if (ks + 1 < KS) load(ks + 1);
        auto frag = [&](const u32x4* s, int part, int blk) {
            return __builtin_bit_cast(bf16x8, s[(part * RB + blk) * 64 + lane]);
        };
        bf16x8 b[WN][3];
#pragma unroll
        for (int j = 0; j < WN; ++j)
#pragma unroll
            for (int p = 0; p < 3; ++p) b[j][p] = frag(sb, p, bn + j);
#pragma unroll
        for (int i = 0; i < WM; ++i) {
            bf16x8 a[3];
#pragma unroll
            for (int p = 0; p < 3; ++p) a[p] = frag(sa, p, am + i);
            // small products first
            constexpr int PA6[6] = {2, 0, 1, 1, 0, 0}, PB6[6] = {0, 2, 1, 0, 1, 0};
#pragma unroll
            for (int t = 0; t < 6; ++t)
#pragma unroll
                for (int j = 0; j < WN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[PA6[t]], b[j][PB6[t]], acc[i][j], 0, 0, 0);
        }
        if (ks + 1 < KS) store((ks + 1) & 1);
        __syncthreads();
    }
    const int li = lane & 31, lk = lane >> 5;
#pragma unroll
    for (int i = 0; i < WM; ++i)
#pragma unroll
        for (int j = 0; j < WN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int row = tm * T + (am + i) * 32 + 8 * (r >> 2) + 4 * lk + (r & 3);
                const int col = tn * T + (bn + j) * 32 + li;
                if (row < M && col < N) C[(int64_t)row * N + col] = acc[i][j][r];
            }
}

}  // namespace sg

// Parts of K the product is computed in (1: no work memory needed).
static int sg_gemm_parts(int64_t M, int64_t N, int64_t K, int num_cu) {
    const int64_t t128 = ((M + 127) / 128) * ((N + 127) / 128), t64 = ((M + 63) / 64) * ((N + 63) / 64);
    if (K > sg::GBUF_MAX_K || N > sg::GBUF_MAX_N || t128 >= num_cu) return 1;
    // two blocks per CU; a part is at least 128 deep, so that adding the parts stays small beside it
    return (int)std::max<int64_t>(1, std::min<int64_t>((int64_t)num_cu * 2 / t64, K / 128));
}

// Is the product computed on bfloat16 parts, and on tiles of which size (0: no)?
// The parts pay for their making (about 65 us for two 4096 x 4096 matrices) where the product is
// deep enough and its tiles reach four fifths of the CUs: 4096^3 1140 -> 790 us, 2048^3 171 ->
// 128; 1024^3, 64 tiles of 128, stays at 34.
static int gemm_split_tile(int64_t M, int64_t N, int64_t K, int num_cu) {
    if (K < 512 || K > (1 << 24) || M > (1 << 20) || N > (1 << 20)) return 0;
    const int64_t t256 = ((M + 255) / 256) * ((N + 255) / 256), t128 = ((M + 127) / 128) * ((N + 127) / 128);
    return t256 * 10 >= num_cu * 8 ? 256 : t128 * 10 >= num_cu * 8 ? 128 : 0;
}
static size_t gemm_plane_bytes(int64_t rows, int64_t K, int T) {
    return (size_t)((rows + T - 1) / T * T) * (size_t)((K + sg::SK - 1) / sg::SK * sg::SK) * 6;
}

// Work memory of the product (bytes; 0: none).  Without it the product runs on the FP32 cores, K
// in one part.
size_t sg_gemm_work_bytes(int64_t M, int64_t N, int64_t K, int num_cu) {
    if (const int T = gemm_split_tile(M, N, K, num_cu)) return 256 + gemm_plane_bytes(M, K, T) + gemm_plane_bytes(N, K, T);
    const int parts = sg_gemm_parts(M, N, K, num_cu);
    return parts > 1 ? (size_t)parts * M * N * 4 : 0;
}

template <int T>
static void launch_split(const float* A, const float* B, float* C, int64_t M, int64_t N, int64_t K, char* work, hipStream_t s) {
    using namespace sg;
    const int KS = (int)((K + SK - 1) / SK);
    uint32_t* flag = (uint32_t*)work;
    u32x4* pa = (u32x4*)(work + 256);
    u32x4* pb = (u32x4*)(work + 256 + gemm_plane_bytes(M, K, T));
    hipLaunchKernelGGL(gemm_flag_kernel, dim3(1), dim3(1), 0, s, flag);
    const unsigned gx = (unsigned)((KS + 7) / 8);
    hipLaunchKernelGGL((gemm_split_kernel<T, false>), dim3(gx, (unsigned)((M + T - 1) / T * (T / 32))), dim3(256), 0, s, A, pa,
                       (int)M, (int)K, K, KS, flag);
    hipLaunchKernelGGL((gemm_split_kernel<T, true>), dim3(gx, (unsigned)((N + T - 1) / T * (T / 32))), dim3(256), 0, s, B, pb,
                       (int)N, (int)K, N, KS, flag);
    hipLaunchKernelGGL((gemm_parts_kernel<T, 8>), dim3((unsigned)(((M + T - 1) / T) * ((N + T - 1) / T))), dim3(64 * 8), 0, s, pa, pb, C,
                       (int)M, (int)N, KS, flag);
}

// work: sg_gemm_work_bytes(), or null.
hipError_t sg_launch_gemm_f32(const float* A, const float* B, float* C, int64_t M, int64_t N, int64_t K, int num_cu,
                              void* work, hipStream_t s) {
    if (M <= 0 || N <= 0) return hipSuccess;
    if (M > (1 << 30) || N > (1 << 30) || K > (1 << 30)) return hipErrorInvalidValue;
    const int64_t t128 = ((M + 127) / 128) * ((N + 127) / 128), t64 = ((M + 63) / 64) * ((N + 63) / 64);
    if (t64 > (1 << 30)) return hipErrorInvalidValue;
    const uint32_t* only_if = nullptr;
    const int split = work ? gemm_split_tile(M, N, K, num_cu) : 0;
    if (split == 256) launch_split<256>(A, B, C, M, N, K, (char*)work, s);
    else if (split == 128) launch_split<128>(A, B, C, M, N, K, (char*)work, s);
    if (split) only_if = (const uint32_t*)work;  // the FP32 kernel runs if the parts would not do
    const int parts = split || !work ? 1 : sg_gemm_parts(M, N, K, num_cu);
    float* out = parts > 1 ? (float*)work : C;
    int64_t kpart = (K + parts - 1) / parts;
    kpart = std::max<int64_t>(1, parts > 1 ? (kpart + 31) / 32 * 32 : K);
    if (K > sg::GBUF_MAX_K || N > sg::GBUF_MAX_N)
        hipLaunchKernelGGL((sg::gemm_f32_kernel<128, 16, 1, true>), dim3((unsigned)t128), dim3(256), 0, s, A, B, out, (int)M,
                           (int)N, (int)K, (int)kpart, only_if);
    else if (t128 >= num_cu)
        hipLaunchKernelGGL((sg::gemm_f32_kernel<128, 16, 1>), dim3((unsigned)t128), dim3(256), 0, s, A, B, out, (int)M, (int)N,
                           (int)K, (int)kpart, only_if);
    else
        hipLaunchKernelGGL((sg::gemm_f32_kernel<64, 32, 2>), dim3((unsigned)t64, (unsigned)std::max<int64_t>(1, (K + kpart - 1) / kpart)), dim3(256),
                           0, s, A, B, out, (int)M, (int)N, (int)K, (int)kpart, only_if);
    if (parts > 1)
        hipLaunchKernelGGL(sg::gemm_sum_kernel, dim3((unsigned)((M * N + 255) / 256)), dim3(256), 0, s, (const float*)work, C, M * N,
                           (int)((K + kpart - 1) / kpart));
    return hipGetLastError();
}
