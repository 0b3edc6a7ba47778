// Matrix transposition and matrix-vector products (Section 3.4: transpose, right_multiply,
// left_multiply; Listing 1).  Both read and write HBM once per element, so they are built for
// bandwidth: the transpose moves 64 x 64 tiles through LDS (coalesced 16-byte reads of rows,
// coalesced 16-byte writes of the transposed rows, 4-byte accesses in tiles at the matrix's
// edge or with unaligned rows, a padded tile against bank conflicts); the right product gives
// each row a wave (four waves where the rows are few), the left product gives each block 256
// columns of a chunk of rows, its waves taking every fourth row, and a second kernel adds the
// chunks.  Loads are 16 bytes at any alignment, eight in flight per lane, and every sum has a
// fixed order: float64 sums of exact float32 products, rounded to float32, identical from run
// to run.  10,000 x 8192: right 57 us (5.7 TB/s; 61 with one load in flight), left 53 + 5 us
// (6.2 TB/s; 86 + 17 with 4-byte loads and one thread adding all the chunks of a column).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "sg_runtime.h"

namespace sgl {

constexpr int TT = 64;  // transpose tile

// Do the values fail a check?  Not finite: the bits reach 0x7F800000 as a signed integer (+inf,
// positive NaNs) or 0xFF800000 as an unsigned one (-inf, negative NaNs).
template <int K>
__device__ __forceinline__ bool fails(const sgrt::FusedCheck& chk, const uint32_t (&x)[K]) {
    bool bad = false;
    for (int i = 0; i < chk.n; ++i) {
        const sg::SgOp& op = chk.ops[i];
        if (op.pad == sg::P_FINITE) {
            int32_t ms = INT32_MIN;
            uint32_t mu = 0u;
#pragma unroll
            for (int k = 0; k < K; ++k) {
                ms = max(ms, (int32_t)x[k]);
                mu = max(mu, x[k]);
            }
            bad |= ms >= 0x7F800000 || mu >= 0xFF800000u;
        } else if (op.pad == sg::P_RANGE_F) {
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const float f = __builtin_bit_cast(float, x[k]);
                bad |= !(f >= op.c0.f && f <= op.c1.f);
            }
        } else {
#pragma unroll
            for (int k = 0; k < K; ++k) bad |= (int32_t)x[k] < op.c0.i || (int32_t)x[k] > op.c1.i;
        }
    }
    return bad;
}

// CHECK: the contract's predicates are evaluated on the elements as they pass, so that the
// contract's own pass reads the result again only when one fails (to find the first).
template <bool CHECK>
__global__ __launch_bounds__(256) void t_transpose(const uint32_t* __restrict__ a, uint32_t* __restrict__ b,
                                                   int64_t rows, int64_t cols, const sgrt::FusedCheck chk) {
    __shared__ uint32_t tile[TT][TT + 1];
    auto report = [&](bool bad) {
        if (__ballot(bad) && (threadIdx.x & 63) == 0)
            __hip_atomic_store(chk.flag, (uint64_t)1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    const int64_t r0 = (int64_t)blockIdx.y * TT, c0 = (int64_t)blockIdx.x * TT;
    // a tile inside the matrix with 16-byte aligned rows: 16-byte reads of 16 rows and 16-byte
    // writes of 16 transposed rows per step (the same for the whole block)
    if (r0 + TT <= rows && c0 + TT <= cols && rows % 4 == 0 && cols % 4 == 0 &&
        ((reinterpret_cast<uintptr_t>(a) | reinterpret_cast<uintptr_t>(b)) & 15) == 0) {
        const int tr = threadIdx.x >> 4, tc = (threadIdx.x & 15) * 4;
        uint4 v[TT / 16];
#pragma unroll
        for (int k = 0; k < TT / 16; ++k) v[k] = *reinterpret_cast<const uint4*>(a + (r0 + tr + 16 * k) * cols + c0 + tc);
#pragma unroll
        for (int k = 0; k < TT / 16; ++k) {
            uint32_t* t = &tile[tr + 16 * k][tc];
            t[0] = v[k].x; t[1] = v[k].y; t[2] = v[k].z; t[3] = v[k].w;
        }
        if (CHECK) {
            uint32_t x[TT / 4];
#pragma unroll
            for (int k = 0; k < TT / 16; ++k) {
                x[4 * k + 0] = v[k].x; x[4 * k + 1] = v[k].y; x[4 * k + 2] = v[k].z; x[4 * k + 3] = v[k].w;
            }
            report(fails(chk, x));
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < TT / 16; ++k) {
            const int c = tr + 16 * k;  // output row c0 + c, columns r0 + tc .. + 3
            uint4 o;
            o.x = tile[tc + 0][c]; o.y = tile[tc + 1][c]; o.z = tile[tc + 2][c]; o.w = tile[tc + 3][c];
            *reinterpret_cast<uint4*>(b + (c0 + c) * rows + r0 + tc) = o;
        }
        return;
    }
    const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;  // 64 x 4 threads
    // places outside the matrix take the tile's first element, which is checked with the others:
    // loads and check without a condition around each (10^6 x 1 with its check 91 -> 59 us)
    const uint32_t first = a[r0 * cols + c0];
    uint32_t x[TT / 4];
#pragma unroll
    for (int k = 0; k < TT / 4; ++k) {
        const int64_t r = r0 + ty + 4 * k, c = c0 + tx;
        x[k] = r < rows && c < cols ? a[r * cols + c] : first;
    }
#pragma unroll
    for (int k = 0; k < TT / 4; ++k) tile[ty + 4 * k][tx] = x[k];
    if (CHECK) report(fails(chk, x));
    __syncthreads();
#pragma unroll
    for (int k = 0; k < TT / 4; ++k) {
        const int64_t c = c0 + ty + 4 * k, r = r0 + tx;  // output row c, column r
        if (r < rows && c < cols) b[c * rows + r] = tile[tx][ty + 4 * k];
    }
}

// 16 bytes at the 4-byte alignment that every float array has
typedef float f4 __attribute__((ext_vector_type(4), aligned(4)));

// A float32 product is exact in float64, so the fused operation rounds as the sum alone does.
__device__ __forceinline__ double fma4(const f4 a, const f4 b, double acc) {
    acc = __builtin_fma((double)a.x, (double)b.x, acc);
    acc = __builtin_fma((double)a.y, (double)b.y, acc);
    acc = __builtin_fma((double)a.z, (double)b.z, acc);
    return __builtin_fma((double)a.w, (double)b.w, acc);
}

// y = M v: WPR waves per row, each over every WPR-th stretch of 4 x 256 columns
template <int WPR>
__global__ __launch_bounds__(256) void mv_right(const float* __restrict__ M, const float* __restrict__ v,
                                                float* __restrict__ y, int64_t rows, int64_t cols) {
    __shared__ double part[4];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t row = WPR == 1 ? (int64_t)blockIdx.x * 4 + wave : (int64_t)blockIdx.x;
    if (row >= rows) return;  // the whole block where it has a barrier
    const float* m = M + row * cols;
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    int64_t k = (int64_t)(WPR == 1 ? 0 : wave) * 1024;
    for (; k + 1024 <= cols; k += 1024 * WPR) {
        f4 a[4], b[4];  // eight 16-byte loads in flight
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            a[q] = *reinterpret_cast<const f4*>(m + k + q * 256 + lane * 4);
            b[q] = *reinterpret_cast<const f4*>(v + k + q * 256 + lane * 4);
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) acc[q] = fma4(a[q], b[q], acc[q]);
    }
    // the stretch that the row's end cuts belongs to one wave: its loads are issued together too
    // (places past the end read the row's last four columns and count as zero)
    if (k < cols && (WPR == 1 || k / 1024 % WPR == wave)) {
        if (cols >= 4) {
            f4 a[4], b[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                if (k + q * 256 >= cols) break;  // (the same for the whole wave)
                const int64_t c = std::min<int64_t>(k + q * 256 + lane * 4, cols - 4);
                a[q] = *reinterpret_cast<const f4*>(m + c);
                b[q] = *reinterpret_cast<const f4*>(v + c);
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                if (k + q * 256 >= cols) break;
                const bool in = k + q * 256 + lane * 4 + 4 <= cols;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    a[q][e] = in ? a[q][e] : 0.f;
                    b[q][e] = in ? b[q][e] : 0.f;
                }
                acc[q] = fma4(a[q], b[q], acc[q]);
            }
        }
        const int64_t j = cols / 4 * 4 + lane;
        if (j < cols) acc[0] = __builtin_fma((double)m[j], (double)v[j], acc[0]);
    }
    double s = (acc[0] + acc[1]) + (acc[2] + acc[3]);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
    if (WPR == 1) {
        if (lane == 0) y[row] = (float)s;
        return;
    }
    if (lane == 0) part[wave] = s;
    __syncthreads();
    if (threadIdx.x == 0) y[row] = (float)((part[0] + part[1]) + (part[2] + part[3]));
}

// y = M v for rows of at most 512 columns: 16 lanes a row, four columns a lane and step.  A wave per row
// leaves most lanes idle: 10^6 x 1 162 -> 41 us, 100000 x 65 35 -> 18, 20000 x 500 21 -> 19 (1000 columns 24 -> 27).
__global__ __launch_bounds__(256) void mv_right_narrow(const float* __restrict__ M, const float* __restrict__ v,
                                                       float* __restrict__ y, int64_t rows, int64_t cols) {
    const int64_t row = (int64_t)blockIdx.x * 16 + (threadIdx.x >> 4);
    const float* m = M + row * cols;
    double s = 0.0;
    for (int64_t c = (threadIdx.x & 15) * 4; c < cols && row < rows; c += 64) {
        if (c + 4 <= cols) s = fma4(*reinterpret_cast<const f4*>(m + c), *reinterpret_cast<const f4*>(v + c), s);
        else
            for (int64_t j = c; j < cols; ++j) s = __builtin_fma((double)m[j], (double)v[j], s);
    }
#pragma unroll
    for (int o = 8; o > 0; o >>= 1) s += __shfl_xor(s, o);
    if (row < rows && (threadIdx.x & 15) == 0) y[row] = (float)s;
}

// partial[chunk][j] = sum over the chunk's rows of v_i M[i][j]: 256 columns per block, four per
// lane, a wave for every fourth row of the chunk
__global__ __launch_bounds__(256) void mv_left_part(const float* __restrict__ M, const float* __restrict__ v,
                                                    double* __restrict__ part, float* __restrict__ y, int64_t rows,
                                                    int64_t cols, int64_t rows_per_chunk) {
    __shared__ double ws[3][256];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t j = (int64_t)blockIdx.x * 256 + lane * 4;
    const int64_t i0 = (int64_t)blockIdx.y * rows_per_chunk, i1 = std::min<int64_t>(rows, i0 + rows_per_chunk);
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    int64_t i = i0 + wave;
    if (j + 4 <= cols) {
        auto add = [&](const f4 m, float x) {
            acc[0] = __builtin_fma((double)x, (double)m.x, acc[0]);
            acc[1] = __builtin_fma((double)x, (double)m.y, acc[1]);
            acc[2] = __builtin_fma((double)x, (double)m.z, acc[2]);
            acc[3] = __builtin_fma((double)x, (double)m.w, acc[3]);
        };
        for (; i + 28 < i1; i += 32) {  // eight rows in flight per wave
            f4 m[8];
            float x[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                m[q] = *reinterpret_cast<const f4*>(M + (i + 4 * q) * cols + j);
                x[q] = v[i + 4 * q];
            }
#pragma unroll
            for (int q = 0; q < 8; ++q) add(m[q], x[q]);
        }
        for (; i < i1; i += 4) add(*reinterpret_cast<const f4*>(M + i * cols + j), v[i]);
    } else {
        for (; i < i1; i += 4)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (j + q < cols) acc[q] = __builtin_fma((double)v[i], (double)M[i * cols + j + q], acc[q]);
    }
    if (wave > 0)
#pragma unroll
        for (int q = 0; q < 4; ++q) ws[wave - 1][lane * 4 + q] = acc[q];
    __syncthreads();
    if (wave == 0)
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (j + q < cols) {
                const double s = (acc[q] + ws[0][lane * 4 + q]) + (ws[1][lane * 4 + q] + ws[2][lane * 4 + q]);
                if (y) y[j + q] = (float)s;  // a single chunk: nothing to add
                else part[(int64_t)blockIdx.y * cols + j + q] = s;
            }
}

// y = the chunks' sums: 32 columns per block, a thread for every eighth of the chunks (in order,
// then the eighths in order)
__global__ __launch_bounds__(256) void mv_left_sum(const double* __restrict__ part, float* __restrict__ y,
                                                   int64_t cols, int64_t chunks) {
    __shared__ double ws[8][32];
    const int c = threadIdx.x & 31, g = threadIdx.x >> 5;
    const int64_t j = (int64_t)blockIdx.x * 32 + c;
    const int64_t per = (chunks + 7) / 8, c0 = g * per, c1 = std::min<int64_t>(chunks, c0 + per);
    double acc = 0.0;
    if (j < cols) {
#pragma unroll 8
        for (int64_t k = c0; k < c1; ++k) acc += part[k * cols + j];
    }
    ws[g][c] = acc;
    __syncthreads();
    if (g != 0 || j >= cols) return;
#pragma unroll
    for (int k = 1; k < 8; ++k) acc += ws[k][c];
    y[j] = (float)acc;
}

}  // namespace sgl

namespace sgrt {

sg_status run_linalg(sg_ctx_s* ctx, sg_node_s* n, const FusedCheck* check) {
    using namespace sgl;
    hipStream_t st = ctx->stream;
    if (n->op == OPN_TRANSPOSE) {
        const sg_node_s* a = n->src[0];
        const int64_t rows = a->rows, cols = a->cols;
        if (rows > 0 && cols > 0) {
            const dim3 grid((unsigned)((cols + TT - 1) / TT), (unsigned)((rows + TT - 1) / TT));
            if (check)
                hipLaunchKernelGGL(t_transpose<true>, grid, dim3(256), 0, st, (const uint32_t*)a->dev, (uint32_t*)n->dev, rows,
                                   cols, *check);
            else
                hipLaunchKernelGGL(t_transpose<false>, grid, dim3(256), 0, st, (const uint32_t*)a->dev, (uint32_t*)n->dev, rows,
                                   cols, FusedCheck());
            SG_HIP(ctx, hipGetLastError());
        }
        n->count = n->n;
        return SG_OK;
    }
    if (n->op != OPN_MATVEC) return fail(ctx, SG_E_INVALID, "run_linalg: not a transpose or matrix-vector product");
    const sg_node_s* M = n->src[0];
    const sg_node_s* v = n->src[1];
    const int64_t rows = M->rows, cols = M->cols;
    n->count = n->n;
    if (n->binop == 0) {  // right: y = M v
        if (rows == 0) return SG_OK;
        // a wave per row, four where that would leave CUs without a block, a quarter for short rows
        if (cols <= 512 && rows >= 16 * (int64_t)ctx->num_cu)
            hipLaunchKernelGGL(mv_right_narrow, dim3((unsigned)((rows + 15) / 16)), dim3(256), 0, st, (const float*)M->dev,
                               (const float*)v->dev, (float*)n->dev, rows, cols);
        else if (rows >= 4 * (int64_t)ctx->num_cu * 4)
            hipLaunchKernelGGL(mv_right<1>, dim3((unsigned)((rows + 3) / 4)), dim3(256), 0, st, (const float*)M->dev,
                               (const float*)v->dev, (float*)n->dev, rows, cols);
        else
            hipLaunchKernelGGL(mv_right<4>, dim3((unsigned)rows), dim3(256), 0, st, (const float*)M->dev, (const float*)v->dev,
                               (float*)n->dev, rows, cols);
        SG_HIP(ctx, hipGetLastError());
        return SG_OK;
    }
    // left: y = v M, rows split into chunks so that the grid fills the device
    if (cols == 0) return SG_OK;
    const int64_t cblocks = (cols + 255) / 256;
    const int64_t chunks = std::max<int64_t>(1, std::min<int64_t>((rows + 31) / 32, (2048 + cblocks - 1) / cblocks));
    const int64_t rpc = std::max<int64_t>(1, (rows + chunks - 1) / chunks);
    const int64_t nch = std::max<int64_t>(1, (rows + rpc - 1) / rpc);
    float* y = rows > 0 && nch == 1 ? (float*)n->dev : nullptr;
    double* part = y ? nullptr : (double*)dev_alloc(ctx, (size_t)nch * cols * sizeof(double));
    if (!part && !y) return fail(ctx, SG_E_OOM, "left_multiply: workspace");
    if (rows > 0) {
        hipLaunchKernelGGL(mv_left_part, dim3((unsigned)cblocks, (unsigned)nch), dim3(256), 0, st, (const float*)M->dev,
                           (const float*)v->dev, part, y, rows, cols, rpc);
    } else {
        (void)hipMemsetAsync(part, 0, (size_t)cols * sizeof(double), st);
    }
    hipError_t e = hipGetLastError();
    if (e == hipSuccess && !y) {
        hipLaunchKernelGGL(mv_left_sum, dim3((unsigned)((cols + 31) / 32)), dim3(256), 0, st, part, (float*)n->dev, cols,
                           rows > 0 ? nch : 1);
        e = hipGetLastError();
    }
    if (part) dev_free(ctx, part);  // handed out again in stream order only
    if (e != hipSuccess) return hip_fail(ctx, e, "left_multiply");
    return SG_OK;
}

}  // namespace sgrt
