// Determinant by Gaussian elimination (Section 5, Listing 5): a loop of fused row updates,
// captured once into a HIP graph and replayed.
//
// The listing's inner loop is the row update of the optimizer's example: every row below the
// pivot row loses a multiple of it, fused into one expression per element.  The elimination
// here is the textbook one (partial pivoting; a zero pivot means the matrix is singular), in
// float64 on the float32 input widened exactly.  Up to 4096 rows it runs by panels of columns,
// a workgroup per panel and a kernel for the columns behind it; beyond, per column k: one block finds the pivot row
// (largest |W[i][k]|, the first on ties, NaN largest) and multiplies it into the determinant;
// a swap kernel exchanges the pivot row with row k; the update kernel computes
// W[i][j] = W[i][j] - (W[i][k] / W[k][k]) * W[k][j] for the trailing block, the multiplier once
// per row in LDS, the product and the difference rounded separately (no fused multiply-add).
// The determinant is kept as sign, mantissa in [0.5, 1) and binary exponent, so it is exact to
// the last rounding even where it leaves the float64 range.  The kernels are captured into one
// graph per node (and per buffer address), replayed by every later execution.
#include <hip/hip_runtime.h>

#include <cmath>
#include <string>

#include "sg_runtime.h"

namespace sgg {

constexpr int GB = 256;  // threads per block
constexpr int GR = 8;    // rows per update block

struct DetState {
    int32_t sign;      // -1, 1; 0 once singular
    int32_t singular;
    int64_t expo;      // det = sign * mant * 2^expo
    double mant;       // in [0.5, 1)
    int64_t piv;       // pivot row of the current column
};

__global__ void g_init(const float* __restrict__ A, double* __restrict__ W, int64_t nn, int32_t* __restrict__ rowmap,
                       int32_t n, DetState* st) {
    const int64_t i = (int64_t)blockIdx.x * GB + threadIdx.x;
    if (i < nn) W[i] = (double)A[i];
    if (rowmap && i < n) rowmap[i] = (int32_t)i;
    if (i == 0) {
        st->sign = 1;
        st->singular = 0;
        st->expo = 1;  // the empty product: 1 = 0.5 * 2^1
        st->mant = 0.5;
        st->piv = 0;
    }
}

// order of |x| as an unsigned key: |x| bit patterns are monotone, NaN above infinity
__device__ __forceinline__ uint64_t abs_key(double x) {
    return __builtin_bit_cast(uint64_t, x) & 0x7FFFFFFFFFFFFFFFull;
}

__global__ __launch_bounds__(GB) void g_pivot(double* __restrict__ W, int64_t n, int64_t k, DetState* st) {
    __shared__ uint64_t skey[GB / 64];
    __shared__ int64_t sidx[GB / 64];
    if (st->singular) return;
    uint64_t best = 0;
    int64_t bi = k;
    for (int64_t i = k + threadIdx.x; i < n; i += GB) {
        const uint64_t key = abs_key(W[i * n + k]);
        if (key > best) { best = key; bi = i; }  // rows in increasing order: ties keep the first
    }
    if (best == 0) bi = n;  // no nonzero entry seen by this thread
    for (int o = 32; o > 0; o >>= 1) {
        const uint64_t kb = __shfl_xor(best, o);
        const int64_t ib = __shfl_xor(bi, o);
        if (kb > best || (kb == best && ib < bi)) { best = kb; bi = ib; }
    }
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (lane == 0) { skey[wave] = best; sidx[wave] = bi; }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < GB / 64; ++w)
            if (skey[w] > best || (skey[w] == best && sidx[w] < bi)) { best = skey[w]; bi = sidx[w]; }
        if (best == 0) {  // the column is zero from row k down: singular
            st->singular = 1;
            st->sign = 0;
            st->mant = 0.0;
            st->expo = 0;
            return;
        }
        const double piv = W[bi * n + k];
        int pe = 0;
        double pm = frexp(piv, &pe);
        int32_t sg = st->sign * (bi != k ? -1 : 1);
        if (pm < 0) { pm = -pm; sg = -sg; }
        int e2 = 0;
        const double m = frexp(st->mant * pm, &e2);
        st->mant = m;
        st->expo += (int64_t)pe + e2;
        st->sign = sg;
        st->piv = bi;
    }
}

__global__ __launch_bounds__(GB) void g_swap(double* __restrict__ W, int64_t n, int64_t k, const DetState* st) {
    if (st->singular) return;
    const int64_t p = st->piv;
    if (p == k) return;
    const int64_t j = k + (int64_t)blockIdx.x * GB + threadIdx.x;
    if (j < n) {
        const double a = W[k * n + j], b = W[p * n + j];
        W[k * n + j] = b;
        W[p * n + j] = a;
    }
}

__global__ __launch_bounds__(GB) void g_update(double* __restrict__ W, int64_t n, int64_t k, const DetState* st) {
    __shared__ double l[GR];
    if (st->singular) return;
    const int64_t i0 = k + 1 + (int64_t)blockIdx.y * GR;
    const int64_t j = k + 1 + (int64_t)blockIdx.x * GB + threadIdx.x;
    if (threadIdx.x < GR) {
        const int64_t i = i0 + threadIdx.x;
        l[threadIdx.x] = i < n ? W[i * n + k] / W[k * n + k] : 0.0;
    }
    __syncthreads();
    if (j >= n) return;
    const double pk = W[k * n + j];
#pragma unroll
    for (int r = 0; r < GR; ++r) {
        const int64_t i = i0 + r;
        if (i < n) {
            const double prod = l[r] * pk;
            W[i * n + j] = W[i * n + j] - prod;
        }
    }
}

// ---- elimination by panels (n <= GPANEL_MAX) -------------------------------------------------
//
// A column of the elimination needs the one before it: n steps of pivot search, exchange and
// update.  As kernels of a graph a step costs three launches, about 10 us (n = 1000: 9.96 ms; by
// panels 1.76 ms, two thirds of it in g_panel).  Here one workgroup runs the steps of a panel of NB columns with the panel's rows in
// registers (R rows per thread) and two barriers per column: every wave picks the pivot among
// the waves' candidates, then its row goes through LDS.  Rows are not moved: a thread's row carries its
// logical position, and `rowmap` maps positions to rows of W.  Then one kernel applies the
// panel's NB updates to the trailing columns, a thread per column: first to the pivot rows
// themselves (in registers), then to its rows.  Every element sees the same products and
// differences in the same order as column by column (each rounded), so the determinant is the
// same to the last bit.

constexpr int GPANEL = 16;        // columns of a panel
constexpr int GPANEL_MAX = 4096;  // rows that one workgroup's registers hold (4 per thread)

__device__ __forceinline__ uint32_t dpp_max(uint32_t v, bool row_only) {
    // identity 0; lane 15 ends with the maximum of the first 16 lanes, lane 63 with the wave's
#define SGG_STEP(CTRL, ROWS) v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWS, 0xF, false))
    SGG_STEP(0x111, 0xF);  // row_shr:1
    SGG_STEP(0x112, 0xF);  // row_shr:2
    SGG_STEP(0x114, 0xF);  // row_shr:4
    SGG_STEP(0x118, 0xF);  // row_shr:8
    if (row_only) return (uint32_t)__builtin_amdgcn_readlane((int)v, 15);
    SGG_STEP(0x142, 0xA);  // row_bcast:15
    SGG_STEP(0x143, 0xC);  // row_bcast:31
#undef SGG_STEP
    return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

// The lane holding the largest key, the lowest position among equal ones; -1 when every key is
// zero.  For the rare column whose largest high words tie.
__device__ int wave_pick(uint64_t key, int32_t pos) {
    const uint32_t hi = (uint32_t)(key >> 32), lo = (uint32_t)key;
    // every lane takes part in each reduction
    const uint32_t mh = dpp_max(hi, false);
    const bool in = hi == mh && key != 0;
    const uint32_t ml = dpp_max(in ? lo : 0u, false);
    const bool in2 = in && lo == ml;
    const uint32_t first = in2 ? 0x7FFFFFFFu - (uint32_t)pos : 0u;
    const uint32_t mf = dpp_max(first, false);
    const uint64_t cand = __ballot(in2 && first == mf);
    return cand ? __builtin_ctzll(cand) : -1;
}

// Multipliers go to L[k][row of W] for the trailing update.  The current column is always a
// row's first register: the update of column j writes register j - 1, so one loop body (no
// register indexed by k) serves every column.  A column takes about 2000 cycles, a chain of
// latencies: the wave's candidate (a maximum over the high words of |x| by data-parallel shifts,
// whose lane is found by ballots), LDS and barrier, the workgroup's pivot, then the division of
// the rows while the pivot row goes through LDS, then the update.
template <int R, int NB, int MAXT>
__global__ __launch_bounds__(MAXT) void g_panel(const double* __restrict__ W, double* __restrict__ L, int n, int k0, int nb,
                                                int32_t* __restrict__ rowmap, double* __restrict__ pivots,
                                                int32_t* __restrict__ moved, DetState* __restrict__ st) {
    __shared__ double tile[MAXT / 64][64][NB + 1];
    __shared__ double prow[NB];
    __shared__ uint64_t sval[2][64];
    __shared__ int32_t spos[2][64];
    if (st->singular) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, B = blockDim.x, nw = B >> 6;
    double a[R][NB];
    int32_t pos[R], row[R];
    // 64 rows at a time through LDS: the wave's loads run along the rows' NB columns
#pragma unroll
    for (int q = 0; q < R; ++q) {
        pos[q] = k0 + tid + q * B;
        row[q] = pos[q] < n ? rowmap[pos[q]] : -1;
        if (pos[q] >= n) pos[q] = -1;  // never a candidate, never updated
    }
#pragma unroll
    for (int q = 0; q < R; ++q) {
        double x[NB];
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            const int r = (i * 64 + lane) / NB, c = lane % NB;
            const int32_t rr = __shfl(row[q], r);
            x[i] = rr >= 0 && c < nb ? W[(int64_t)rr * n + k0 + c] : 0.0;
        }
#pragma unroll
        for (int i = 0; i < NB; ++i) tile[wave][(i * 64 + lane) / NB][lane % NB] = x[i];
#pragma unroll
        for (int j = 0; j < NB; ++j) a[q][j] = tile[wave][lane][j];
    }
#pragma unroll 1
    for (int k = 0; k < nb; ++k) {
        const int buf = k & 1, kp = k0 + k;
        // the wave's candidate; rows chosen already lie at positions below kp
        uint32_t hi[R], hmax = 0;
#pragma unroll
        for (int q = 0; q < R; ++q) {
            hi[q] = pos[q] >= kp ? (uint32_t)(abs_key(a[q][0]) >> 32) : 0u;
            hmax = max(hmax, hi[q]);
        }
        const uint32_t mh = dpp_max(hmax, false);
        int wq = 0, wl = -1, ncand = 0;
#pragma unroll
        for (int q = 0; q < R; ++q) {
            const uint64_t c = __ballot(hi[q] == mh);
            if (c) { wq = q; wl = __builtin_ctzll(c); }
            ncand += __builtin_popcountll(c);
        }
        if (__builtin_expect(mh == 0 || ncand != 1, 0)) {
            uint64_t key = 0;
            int32_t kpos = 0;
            int kq = 0;
#pragma unroll
            for (int q = 0; q < R; ++q) {
                const uint64_t x = pos[q] >= kp ? abs_key(a[q][0]) : 0;
                if (x > key || (x == key && x != 0 && pos[q] < kpos)) { key = x; kpos = pos[q]; kq = q; }
            }
            wl = wave_pick(key, kpos);
            wq = wl < 0 ? 0 : __builtin_amdgcn_readlane(kq, wl);
        }
        if (lane == (wl < 0 ? 0 : wl)) {
            double v = a[0][0];
            int32_t vp = pos[0];
#pragma unroll
            for (int q = 1; q < R; ++q) {
                v = wq == q ? a[q][0] : v;
                vp = wq == q ? pos[q] : vp;
            }
            sval[buf][wave] = wl < 0 ? 0 : __builtin_bit_cast(uint64_t, v);
            spos[buf][wave] = vp;
        }
        __syncthreads();
        // the workgroup's pivot, picked by every wave from the same values
        const uint64_t val = sval[buf][lane];
        const int32_t vpos = spos[buf][lane];
        const uint64_t vkey = lane < nw ? val & 0x7FFFFFFFFFFFFFFFull : 0;
        const uint32_t vmh = dpp_max((uint32_t)(vkey >> 32), true);
        const uint64_t vc = __ballot(lane < nw && (uint32_t)(vkey >> 32) == vmh);
        int ww = __builtin_ctzll(vc);
        if (__builtin_expect(vmh == 0 || __builtin_popcountll(vc) != 1, 0)) ww = wave_pick(vkey, vpos);
        if (ww < 0) {  // the column is zero from here down: singular (the same for every wave)
            if (tid == 0) {
                st->singular = 1;
                st->sign = 0;
                st->mant = 0.0;
                st->expo = 0;
            }
            return;
        }
        const int32_t pp = __builtin_amdgcn_readlane(vpos, ww);
        const double piv = __builtin_bit_cast(double, ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(val >> 32), ww) << 32) |
                                                          (uint32_t)__builtin_amdgcn_readlane((int)val, ww));
        if (wave == ww) {
#pragma unroll
            for (int q = 0; q < R; ++q)
                if (wq == q && lane == wl) {
#pragma unroll
                    for (int j = 1; j < NB; ++j) prow[j] = a[q][j];
                }
        }
        // the rows' divisions, then their updates, side by side: one wave per SIMD has no other
        // work to cover the latency of a dependent float64 operation
        double l[R];
#pragma unroll
        for (int q = 0; q < R; ++q) {
            pos[q] = pos[q] == pp ? kp : pos[q] == kp ? pp : pos[q];
            l[q] = a[q][0] / piv;
        }
        // a wave one column ahead waits at that column's first barrier before it writes prow
        __syncthreads();
#pragma unroll
        for (int j = 1; j < NB; ++j) {
            const double u = prow[j];
            double prod[R];
#pragma unroll
            for (int q = 0; q < R; ++q) prod[q] = l[q] * u;
#pragma unroll
            for (int q = 0; q < R; ++q) a[q][j - 1] = a[q][j] - prod[q];  // (a pivot row is not read again)
        }
#pragma unroll
        for (int q = 0; q < R; ++q)
            if (pos[q] > kp) L[(int64_t)k * n + row[q]] = l[q];
        if (tid == 0) {
            pivots[kp] = piv;
            moved[kp] = pp != kp;
        }
    }
    // the rows' new positions (every position below n is held by exactly one thread's row: they
    // were only exchanged)
#pragma unroll
    for (int q = 0; q < R; ++q)
        if (pos[q] >= 0) rowmap[pos[q]] = row[q];
}

// The panel's pivots multiplied into the determinant, in column order (the first wave of a
// block; the pivots are loaded side by side, one after another they cost a round trip each).
template <int NB>
__device__ void det_accumulate(const double* pivots, const int32_t* moved, int k0, int nb, DetState* st) {
    const int lane = threadIdx.x;
    const double pv = lane < nb ? pivots[k0 + lane] : 1.0;
    const int mv = lane < nb ? moved[k0 + lane] : 0;
    int32_t sign = st->sign;
    int64_t expo = st->expo;
    double mant = st->mant;
#pragma unroll
    for (int k = 0; k < NB; ++k) {
        int pe = 0, e2 = 0;
        double pm = frexp(__shfl(pv, k), &pe);
        if (k >= nb) break;
        if (__shfl(mv, k)) sign = -sign;
        if (pm < 0) { pm = -pm; sign = -sign; }
        mant = frexp(mant * pm, &e2);
        expo += (int64_t)pe + e2;
    }
    if (lane == 0) {
        st->sign = sign;
        st->expo = expo;
        st->mant = mant;
    }
}

template <int NB>
__global__ __launch_bounds__(64) void g_product(const double* pivots, const int32_t* moved, int k0, int nb, DetState* st) {
    if (st->singular) return;
    det_accumulate<NB>(pivots, moved, k0, nb, st);
}

// Trailing columns of a full panel: a column per lane and 4 * TR rows per block; the last row of
// blocks multiplies the panel's pivots into the determinant meanwhile.  Latency-bound (row
// numbers, rows, multipliers, then the pivot rows' own updates): few rows per wave and many
// blocks.  8.1 us on average over n = 1000 with 4 rows per wave, 9.6 with 8, 17 with 16, 8.6
// with 2; 10.5 and more with two columns per lane.
template <int NB, int TR>
__global__ __launch_bounds__(256) void g_trail(double* __restrict__ W, const double* __restrict__ L, int n, int k0,
                                               const int32_t* __restrict__ rowmap, const double* __restrict__ pivots,
                                               const int32_t* __restrict__ moved, DetState* __restrict__ st) {
    __shared__ double lp[NB][NB];        // multipliers of the pivot rows
    __shared__ double lr[4 * TR][NB];    // and of this block's rows
    __shared__ int32_t prow[NB], rrow[4 * TR];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (blockIdx.y == gridDim.y - 1) {
        if (blockIdx.x == 0 && tid < 64 && !st->singular) det_accumulate<NB>(pivots, moved, k0, NB, st);
        return;
    }
    const int i0 = k0 + NB + (int)blockIdx.y * 4 * TR;
    const int singular = st->singular;
    if (tid < NB) prow[tid] = rowmap[k0 + tid];
    else if (tid >= 64 && tid < 64 + 4 * TR) rrow[tid - 64] = i0 + tid - 64 < n ? rowmap[i0 + tid - 64] : -1;
    if (singular) return;
    __syncthreads();
    const int j = k0 + NB + (int)blockIdx.x * 64 + lane;
    double u[NB], w[TR];
#pragma unroll
    for (int r = 0; r < NB; ++r) u[r] = j < n ? W[(int64_t)prow[r] * n + j] : 0.0;
#pragma unroll
    for (int r = 0; r < TR; ++r) {
        const int32_t i = rrow[wave * TR + r];
        w[r] = i >= 0 && j < n ? W[(int64_t)i * n + j] : 0.0;
    }
    for (int i = tid; i < NB * NB; i += 256) {
        const int r = i % NB, k = i / NB;
        if (k < r) lp[r][k] = L[(int64_t)k * n + prow[r]];
    }
    for (int i = tid; i < 4 * TR * NB; i += 256) {
        const int r = i % (4 * TR), k = i / (4 * TR);
        lr[r][k] = rrow[r] >= 0 ? L[(int64_t)k * n + rrow[r]] : 0.0;
    }
    __syncthreads();
#pragma unroll
    for (int r = 1; r < NB; ++r)
#pragma unroll
        for (int k = 0; k < r; ++k) {
            const double prod = lp[r][k] * u[k];
            u[r] = u[r] - prod;
        }
    // the rows side by side: their chains of dependent differences overlap
#pragma unroll
    for (int k = 0; k < NB; ++k)
#pragma unroll
        for (int r = 0; r < TR; ++r) {
            const double prod = lr[wave * TR + r][k] * u[k];
            w[r] = w[r] - prod;
        }
#pragma unroll
    for (int r = 0; r < TR; ++r) {
        const int32_t i = rrow[wave * TR + r];
        if (i >= 0 && j < n) W[(int64_t)i * n + j] = w[r];
    }
}

// One panel from column k0 on, with as few rows per thread as 512 threads allow: two waves per
// SIMD cover each other's latencies (a panel of 16 columns and 512-1000 rows takes 23 us so, 28
// with four rows in each of 256 threads, 37 and more with a row in each of 1024).  Narrower
// panels only where the rows need 1024 threads.
template <int NB>
void launch_panel(double* W, double* L, int n, int k0, int32_t* rowmap, double* pivots, int32_t* moved, DetState* st,
                  hipStream_t s) {
    const int nb = n - k0 < NB ? n - k0 : NB, rows = n - k0, m = n - k0 - NB;
    auto threads = [&](int per) { return dim3((unsigned)(((rows + per - 1) / per + 63) / 64 * 64)); };
#define SGG_PANEL(R, T) hipLaunchKernelGGL((g_panel<R, NB, T>), dim3(1), threads(R), 0, s, W, L, n, k0, nb, rowmap, pivots, moved, st)
    if constexpr (NB == 8) {
        SGG_PANEL(4, 1024);
    } else {
        if (rows <= 512) SGG_PANEL(1, 512);
        else if (rows <= 1024) SGG_PANEL(2, 512);
        else SGG_PANEL(4, 512);
    }
#undef SGG_PANEL
    if (m > 0)
        hipLaunchKernelGGL((g_trail<NB, 4>), dim3((m + 63) / 64, (m + 15) / 16 + 1), dim3(256), 0, s, W, L, n, k0, rowmap,
                           pivots, moved, st);
    else
        hipLaunchKernelGGL((g_product<NB>), dim3(1), dim3(64), 0, s, pivots, moved, k0, nb, st);
}

hipError_t launch_panels(double* W, double* L, int n, int32_t* rowmap, double* pivots, int32_t* moved, DetState* st,
                         hipStream_t s) {
    for (int k0 = 0; k0 < n;) {
        if (n - k0 > 2048) {
            launch_panel<8>(W, L, n, k0, rowmap, pivots, moved, st, s);
            k0 += 8;
        } else {
            launch_panel<GPANEL>(W, L, n, k0, rowmap, pivots, moved, st, s);
            k0 += GPANEL;
        }
    }
    return hipGetLastError();
}

}  // namespace sgg

namespace sgrt {

// Workspace and captured graph of one determinant node (owned by the node).
struct GaussCache {
    hipGraphExec_t exec = nullptr;
    hipGraph_t graph = nullptr;
    const void* a = nullptr;  // input address the graph was captured for
    void* w = nullptr;        // W (n x n doubles) then the determinant state
    int64_t n = -1;
};

void gauss_cache_free(sg_ctx_s* ctx, void* p) {
    auto* c = (GaussCache*)p;
    if (!c) return;
    if (c->exec) (void)hipGraphExecDestroy(c->exec);
    if (c->graph) (void)hipGraphDestroy(c->graph);
    if (c->w) dev_free(ctx, c->w);
    delete c;
}

sg_status run_gauss(sg_ctx_s* ctx, sg_node_s* node) {
    using namespace sgg;
    sg_node_s* A = node->src[0];
    const int64_t n = A->rows;
    if (A->rows != A->cols) return fail(ctx, SG_E_SHAPE, "determinant: the matrix must be square (rows = columns)");
    if (n > 0 && !A->dev) return fail(ctx, SG_E_STATE, "determinant: matrix has no storage");
    auto* c = (GaussCache*)node->aux;
    if (!c) {
        c = new GaussCache();
        node->aux = c;
    }
    if (c->n != n) {
        if (c->exec) (void)hipGraphExecDestroy(c->exec);
        if (c->graph) (void)hipGraphDestroy(c->graph);
        c->exec = nullptr;
        c->graph = nullptr;
        if (c->w) dev_free(ctx, c->w);
        c->w = dev_alloc(ctx, (size_t)std::max<int64_t>(n * n, 1) * 8 + 512 + (size_t)std::min<int64_t>(n, GPANEL_MAX) * (16 + GPANEL * 8));
        if (!c->w) return fail(ctx, SG_E_OOM, "determinant: workspace");
        c->n = n;
    }
    double* W = (double*)c->w;
    DetState* st = (DetState*)((char*)c->w + (((size_t)std::max<int64_t>(n * n, 1) * 8 + 255) & ~(size_t)255));
    // by panels: a panel's multipliers, pivots, row positions and exchange
    // flags behind the state
    const bool panels = n > 0 && n <= GPANEL_MAX;
    double* L = (double*)((char*)st + 256);
    double* pivots = L + GPANEL * n;
    int32_t* rowmap = (int32_t*)(pivots + n);
    int32_t* moved = rowmap + n;
    if (!c->exec || c->a != A->dev) {
        if (c->exec) (void)hipGraphExecDestroy(c->exec);
        if (c->graph) (void)hipGraphDestroy(c->graph);
        c->exec = nullptr;
        c->graph = nullptr;
        hipStream_t cs = ctx->stream;
        bool own = false;
        if (!cs) {
            SG_HIP(ctx, hipStreamCreate(&cs));
            own = true;
        }
        hipError_t e = hipStreamBeginCapture(cs, hipStreamCaptureModeThreadLocal);
        if (e == hipSuccess) {
            const int64_t nn = n * n;
            hipLaunchKernelGGL(g_init, dim3((unsigned)std::max<int64_t>((nn + GB - 1) / GB, 1)), dim3(GB), 0, cs,
                               (const float*)A->dev, W, nn, panels ? rowmap : nullptr, (int32_t)(panels ? n : 0), st);
            if (panels) e = launch_panels(W, L, (int)n, rowmap, pivots, moved, st, cs);
            for (int64_t k = 0; !panels && k < n && e == hipSuccess; ++k) {
                hipLaunchKernelGGL(g_pivot, dim3(1), dim3(GB), 0, cs, W, n, k, st);
                hipLaunchKernelGGL(g_swap, dim3((unsigned)((n - k + GB - 1) / GB)), dim3(GB), 0, cs, W, n, k, st);
                const int64_t m = n - k - 1;
                if (m > 0)
                    hipLaunchKernelGGL(g_update, dim3((unsigned)((m + GB - 1) / GB), (unsigned)((m + GR - 1) / GR)),
                                       dim3(GB), 0, cs, W, n, k, st);
                e = hipGetLastError();
            }
        }
        hipError_t e2 = hipStreamEndCapture(cs, &c->graph);
        if (own) (void)hipStreamDestroy(cs);
        if (e != hipSuccess || e2 != hipSuccess) return hip_fail(ctx, e != hipSuccess ? e : e2, "determinant: graph capture");
        SG_HIP(ctx, hipGraphInstantiate(&c->exec, c->graph, nullptr, nullptr, 0));
        c->a = A->dev;
    }
    SG_HIP(ctx, hipGraphLaunch(c->exec, ctx->stream));
    DetState h;
    SG_HIP(ctx, hipMemcpyAsync(&h, st, sizeof(h), hipMemcpyDeviceToHost, ctx->stream));
    SG_HIP(ctx, hipStreamSynchronize(ctx->stream));
    node->det_sign = h.sign;
    node->det_mant = h.mant;
    node->det_expo = h.expo;
    const double v = h.mant == 0.0 ? 0.0 : std::ldexp(h.mant, (int)std::max<int64_t>(std::min<int64_t>(h.expo, 4096), -4096));
    node->fval = h.sign < 0 ? -v : v;
    node->f64 = node->fval;
    node->ival = h.sign;
    return SG_OK;
}

}  // namespace sgrt
