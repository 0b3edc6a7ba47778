// Determinant by Gaussian elimination (Section 5, Listing 5): a loop of fused row updates,
// captured once into a HIP graph and replayed.
//
// The listing's inner loop is the row update of the optimizer's example: every row below the
// pivot row loses a multiple of it, fused into one expression per element.  The elimination
// here is the textbook one (partial pivoting; a zero pivot means the matrix is singular), in
// float64 on the float32 input widened exactly.  Up to 4096 rows it runs by panels of columns,
// one workgroup on a panel while others bring the columns behind it up to date; beyond, per
// column k: one block finds the pivot row
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
    int32_t singular;  // 0, or 1 + a column at or before the zero one (by panels: the panel's first)
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
// panels 1.66 ms).  Here one workgroup runs the steps of a panel of NB columns with the panel's
// rows in registers (R rows per thread) and one barrier per column: the waves leave their
// candidates and the candidates' rows in LDS, and every wave picks the pivot among them.  Rows
// are not moved: a thread's row carries its logical position, and `rowmap` maps positions to rows
// of W.  The panel's NB updates go to the trailing columns a thread per column: first to the pivot
// rows themselves (in registers), then to its rows; up to 2048 rows beside the next panel (g_step).
// Every element sees the same products and differences in the same order as column by column
// (each rounded), so the determinant is the same to the last bit.

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

// A barrier for data in LDS.  __syncthreads() also waits for the wave's global stores, here the
// multipliers that the panel writes and never reads.
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Multipliers go to L[k][row of W] for the trailing update.  The current column is always a
// row's first register: the update of column j writes register j - 1, so one loop body (no
// register indexed by k) serves every column.  A column takes 2000 (one row per thread) to 3000
// cycles, a chain of latencies and of instructions that every wave issues: the wave's candidate (a
// maximum over the high words of |x| by data-parallel shifts, whose lane is found by ballots; it is
// looked for amid the updates of the column before), LDS and barrier, the workgroup's pivot, the
// division of the rows, the update.
//
// BEFORE: the panel's columns still lack the updates of the panel before it (multipliers Lb), which
// are applied on the way into the registers: the pivot rows' own part by 16 lanes into LDS, then
// every row: 5 to 8 us, half of it the reads of S.u (a broadcast takes as long as any LDS read).
// rowmap and rowmap_out may be one array (g_panel): read at the start, written at the end.
template <int R, int NB, int MAXT>
struct PanelLds {
    double tile[MAXT / 64][64][NB + 1];
    double prow[2][MAXT / 64][NB];  // the rows of the waves' candidates
    uint64_t sval[2][64];
    int32_t spos[2][64];
    double u[NB][NB], lp[NB][NB];  // BEFORE: the pivot rows in this panel's columns, their multipliers
};
template <int R, int NB, int MAXT, bool BEFORE>
__device__ __forceinline__ void panel(PanelLds<R, NB, MAXT>& S, const double* __restrict__ W, const double* __restrict__ Lb,
                                      double* __restrict__ L, int n, int k0, int nb, const int32_t* rowmap,
                                      int32_t* rowmap_out, double* __restrict__ pivots,
                                      int32_t* __restrict__ moved, DetState* __restrict__ st) {
    auto& tile = S.tile;
    auto& prow = S.prow;
    auto& sval = S.sval;
    auto& spos = S.spos;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, B = blockDim.x, nw = B >> 6;
    double a[R][NB];
    int32_t pos[R], row[R];
    // All loads are issued together: a workgroup alone on its CU pays each round trip in full.
    constexpr int E = BEFORE ? NB * NB / 64 : 1, G = R == 4 ? 4 : NB;
    const int kb = k0 - NB;
    int32_t er[E];         // BEFORE: element tid + e B of u and lp: the row of W of its pivot row,
    double eu[E], el[E];   // the values
    double l[R][G];        // and the first G multipliers of a row
    if (BEFORE) {
#pragma unroll
        for (int e = 0; e < E; ++e) er[e] = tid + e * B < NB * NB ? rowmap[kb + (tid + e * B) / NB] : -1;
    }
#pragma unroll
    for (int q = 0; q < R; ++q) {
        pos[q] = k0 + tid + q * B;
        row[q] = pos[q] < n ? rowmap[pos[q]] : -1;
        if (pos[q] >= n) pos[q] = -1;  // never a candidate, never updated
    }
    if (BEFORE) {
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int c = (tid + e * B) % NB;
            eu[e] = er[e] >= 0 && c < nb ? W[(int64_t)er[e] * n + k0 + c] : 0.0;
            el[e] = er[e] >= 0 ? Lb[(int64_t)c * n + er[e]] : 0.0;
        }
    }
    // 64 rows at a time through LDS: the wave's loads run along the rows' NB columns
#pragma unroll
    for (int q = 0; q < R; ++q)
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            const int r = (i * 64 + lane) / NB, c = lane % NB;
            const int32_t rr = __shfl(row[q], r);
            a[q][i] = rr >= 0 && c < nb ? W[(int64_t)rr * n + k0 + c] : 0.0;
        }
    auto multipliers = [&](int g) {
#pragma unroll
        for (int q = 0; q < R; ++q)
#pragma unroll
            for (int k = 0; k < G; ++k) l[q][k] = Lb[(int64_t)(g + k) * n + (row[q] >= 0 ? row[q] : 0)];
    };
    if (BEFORE) {
        multipliers(0);
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int r = (tid + e * B) / NB, c = (tid + e * B) % NB;
            if (er[e] >= 0) {
                S.u[r][c] = eu[e];
                S.lp[c][r] = el[e];  // (used where c < r)
            }
        }
    }
#pragma unroll
    for (int q = 0; q < R; ++q) {
#pragma unroll
        for (int i = 0; i < NB; ++i) tile[wave][(i * 64 + lane) / NB][lane % NB] = a[q][i];
#pragma unroll
        for (int j = 0; j < NB; ++j) a[q][j] = tile[wave][lane][j];
    }
    if (BEFORE) {
        lds_barrier();
        if (tid < NB) {
            double u[NB];
#pragma unroll
            for (int r = 0; r < NB; ++r) u[r] = S.u[r][tid];
            // the rows side by side: their chains of dependent differences overlap
#pragma unroll
            for (int k = 0; k < NB - 1; ++k) {
#pragma unroll
                for (int r = k + 1; r < NB; ++r) {
                    const double prod = S.lp[k][r] * u[k];
                    u[r] = u[r] - prod;
                }
                S.u[k + 1][tid] = u[k + 1];
                if (k % 4 == 3)
#pragma unroll
                    for (int r = k + 1; r < NB; ++r) asm volatile("" : "+v"(u[r]));
            }
        }
        lds_barrier();
#pragma unroll
        for (int g = 0; g < NB; g += G) {
            if (g) multipliers(g);
#pragma unroll
            for (int k = 0; k < G; ++k) {
                int at = g + k;
                if (k % (R == 1 ? 4 : 2) == 0) {
                    // the updates so far are done here: the compiler would put them all behind all
                    // the reads of S.u, past the registers
#pragma unroll
                    for (int q = 0; q < R; ++q)
#pragma unroll
                        for (int j = 0; j < NB; ++j) asm volatile("" : "+v"(a[q][j]));
                    asm volatile("" : "+v"(at));
                }
#pragma unroll
                for (int j = 0; j < NB; ++j) {
                    const double u = S.u[at][j];
                    double prod[R];
#pragma unroll
                    for (int q = 0; q < R; ++q) prod[q] = l[q][k] * u;
#pragma unroll
                    for (int q = 0; q < R; ++q) a[q][j] = a[q][j] - prod[q];
                }
            }
        }
    }
    // the wave's candidate for the column at position kp; rows chosen already lie below it
    int wq, wl, ncand;
    uint32_t mh;
    auto search = [&](int kp) {
        uint32_t hi[R], hmax = 0;
#pragma unroll
        for (int q = 0; q < R; ++q) {
            hi[q] = pos[q] >= kp ? (uint32_t)(abs_key(a[q][0]) >> 32) : 0u;
            hmax = max(hmax, hi[q]);
        }
        mh = dpp_max(hmax, false);
        wq = 0, wl = -1, ncand = 0;
#pragma unroll
        for (int q = 0; q < R; ++q) {
            const uint64_t c = __ballot(hi[q] == mh);
            wq = c ? q : wq;
            wl = c ? __builtin_ctzll(c) : wl;
            ncand += __builtin_popcountll(c);
        }
    };
    search(k0);
#pragma unroll 1
    for (int k = 0; k < nb; ++k) {
        const int buf = k & 1, kp = k0 + k;
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
        // its whole row goes with it: the pivot's is there when the pivot is known
        if (lane == (wl < 0 ? 0 : wl)) {
#pragma unroll
            for (int q = 0; q < R; ++q)
                if (wq == q) {
                    asm volatile("; row %0" ::"n"(q));  // else the cases share their writes, through copies of the row
                    sval[buf][wave] = wl < 0 ? 0 : __builtin_bit_cast(uint64_t, a[q][0]);
                    spos[buf][wave] = pos[q];
#pragma unroll
                    for (int j = 1; j < NB; ++j) prow[buf][wave][j] = a[q][j];
                }
        }
        lds_barrier();
        // the workgroup's pivot, picked by every wave from the same values; a wave one column ahead
        // writes the other buffer, and waits at that column's barrier before this one is rewritten
        const uint64_t val = sval[buf][lane];
        const int32_t vpos = spos[buf][lane];
        const uint64_t vkey = lane < nw ? val & 0x7FFFFFFFFFFFFFFFull : 0;
        const uint32_t vmh = dpp_max((uint32_t)(vkey >> 32), true);
        const uint64_t vc = __ballot(lane < nw && (uint32_t)(vkey >> 32) == vmh);
        int ww = __builtin_ctzll(vc);
        if (__builtin_expect(vmh == 0 || __builtin_popcountll(vc) != 1, 0)) ww = wave_pick(vkey, vpos);
        if (ww < 0) {  // the column is zero from here down: singular (the same for every wave)
            if (tid == 0) __hip_atomic_store(&st->singular, k0 + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            return;
        }
        const int32_t pp = __builtin_amdgcn_readlane(vpos, ww);
        const double piv = __builtin_bit_cast(double, ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(val >> 32), ww) << 32) |
                                                          (uint32_t)__builtin_amdgcn_readlane((int)val, ww));
        double u[NB];
#pragma unroll
        for (int j = 1; j < NB; ++j) u[j] = prow[buf][ww][j];
        // the rows' divisions, then their updates, side by side: one wave per SIMD has no other
        // work to cover the latency of a dependent float64 operation.  The next column comes first,
        // so that its search fills the gaps of the others' updates
        double l[R];
#pragma unroll
        for (int q = 0; q < R; ++q) {
            pos[q] = pos[q] == pp ? kp : pos[q] == kp ? pp : pos[q];
            l[q] = a[q][0] / piv;
        }
#pragma unroll
        for (int j = 1; j < NB; ++j) {
            double prod[R];
#pragma unroll
            for (int q = 0; q < R; ++q) prod[q] = l[q] * u[j];
#pragma unroll
            for (int q = 0; q < R; ++q) a[q][j - 1] = a[q][j] - prod[q];  // (a pivot row is not read again)
            if (j == 1) search(kp + 1);
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
        if (pos[q] >= 0) rowmap_out[pos[q]] = row[q];
}

template <int R, int NB, int MAXT>
__global__ __launch_bounds__(MAXT) void g_panel(const double* __restrict__ W, double* __restrict__ L, int n, int k0, int nb,
                                                int32_t* rowmap, double* __restrict__ pivots,
                                                int32_t* __restrict__ moved, DetState* __restrict__ st) {
    __shared__ PanelLds<R, NB, MAXT> S;
    if (st->singular) return;
    panel<R, NB, MAXT, false>(S, W, nullptr, L, n, k0, nb, rowmap, rowmap, pivots, moved, st);
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
    if (!st->singular) {
        det_accumulate<NB>(pivots, moved, k0, nb, st);
    } else if (threadIdx.x == 0) {  // whatever the panels before have multiplied together
        st->sign = 0;
        st->mant = 0.0;
        st->expo = 0;
    }
}

// Trailing columns of a full panel: a column per lane and 4 * TR rows per block; the last row of
// blocks multiplies the panel's pivots into the determinant meanwhile.  Latency-bound (row
// numbers, rows, multipliers, then the pivot rows' own updates): few rows per wave and many
// blocks.  8.1 us on average over n = 1000 with 4 rows per wave, 9.6 with 8, 17 with 16, 8.6
// with 2; 10.5 and more with two columns per lane.
template <int NB, int TR, int MAXW>
struct TrailLds {
    double lp[NB][NB];           // multipliers of the pivot rows
    double lr[MAXW * TR][NB];    // and of this block's rows
    int32_t prow[NB], rrow[MAXW * TR];
};
// Rows from i0 on (TR per wave), columns j0 + lane, of the panel at k0.
template <int NB, int TR, int MAXW>
__device__ __forceinline__ void trail(TrailLds<NB, TR, MAXW>& S, double* __restrict__ W, const double* __restrict__ L, int n,
                                      int k0, int i0, int j0, const int32_t* __restrict__ rowmap) {
    auto& lp = S.lp;
    auto& lr = S.lr;
    auto& prow = S.prow;
    auto& rrow = S.rrow;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int B = MAXW == 4 ? 256 : blockDim.x, rows = B / 64 * TR;  // (four waves always, or as many as there are)
    if (tid < NB) prow[tid] = rowmap[k0 + tid];
    for (int i = tid; i < rows; i += B) rrow[i] = i0 + i < n ? rowmap[i0 + i] : -1;
    __syncthreads();
    const int j = j0 + lane;
    double u[NB], w[TR];
#pragma unroll
    for (int r = 0; r < NB; ++r) u[r] = j < n ? W[(int64_t)prow[r] * n + j] : 0.0;
#pragma unroll
    for (int r = 0; r < TR; ++r) {
        const int32_t i = rrow[wave * TR + r];
        w[r] = i >= 0 && j < n ? W[(int64_t)i * n + j] : 0.0;
    }
    for (int i = tid; i < NB * NB; i += B) {
        const int r = i % NB, k = i / NB;
        if (k < r) lp[r][k] = L[(int64_t)k * n + prow[r]];
    }
    for (int i = tid; i < rows * NB; i += B) {
        const int r = i % rows, k = i / rows;
        lr[r][k] = rrow[r] >= 0 ? L[(int64_t)k * n + rrow[r]] : 0.0;
    }
    __syncthreads();
#pragma unroll
    for (int r = 1; r < NB; ++r) {
#pragma unroll
        for (int k = 0; k < r; ++k) {
            const double prod = lp[r][k] * u[k];
            u[r] = u[r] - prod;
        }
    }
    // the rows side by side: their chains of dependent differences overlap
#pragma unroll
    for (int k = 0; k < NB; ++k) {
#pragma unroll
        for (int r = 0; r < TR; ++r) {
            const double prod = lr[wave * TR + r][k] * u[k];
            w[r] = w[r] - prod;
        }
    }
#pragma unroll
    for (int r = 0; r < TR; ++r) {
        const int32_t i = rrow[wave * TR + r];
        if (i >= 0 && j < n) W[(int64_t)i * n + j] = w[r];
    }
}

template <int NB, int TR>
__global__ __launch_bounds__(256) void g_trail(double* __restrict__ W, const double* __restrict__ L, int n, int k0,
                                               const int32_t* __restrict__ rowmap, const double* __restrict__ pivots,
                                               const int32_t* __restrict__ moved, DetState* __restrict__ st) {
    __shared__ TrailLds<NB, TR, 4> S;
    if (st->singular) return;
    if (blockIdx.y == gridDim.y - 1) {
        if (blockIdx.x == 0 && threadIdx.x < 64) det_accumulate<NB>(pivots, moved, k0, NB, st);
        return;
    }
    trail<NB, TR, 4>(S, W, L, n, k0, k0 + NB + (int)blockIdx.y * 4 * TR, k0 + NB + (int)blockIdx.x * 64, rowmap);
}

// The panel at k0 applied, and the next one eliminated beside it: block 0 takes the next panel's
// columns through both, block 1 multiplies the pivots of the panel at k0 into the determinant, the
// others (ncb columns blocks each) apply it to the columns behind.  The next panel's multipliers
// and row positions go to buffers of their own (L1, rowmap1): the others still read this one's.
// One launch in place of two, and the other columns' update no longer between two panels:
// n = 1000 1.75 -> 1.66 ms, 2000 5.40 -> 4.60.
template <int R, int NB, int MAXT, int TR>
__global__ __launch_bounds__(MAXT) void g_step(double* __restrict__ W, const double* __restrict__ L, double* __restrict__ L1,
                                               int n, int k0, int nb, int ncb, const int32_t* __restrict__ rowmap,
                                               int32_t* __restrict__ rowmap1, double* __restrict__ pivots,
                                               int32_t* __restrict__ moved, DetState* __restrict__ st) {
    __shared__ union Lds {
        PanelLds<R, NB, MAXT> p;
        TrailLds<NB, TR, MAXT / 64> t;
    } S;
    // Only an earlier launch's zero column ends a block here.  Block 0 of this one may find another
    // meanwhile (its mark is k0 + NB + 1), and the waves of a block have to agree: one that left
    // before the barriers would leave the others row numbers that nobody wrote.
    const int32_t zero = __hip_atomic_load(&st->singular, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (zero != 0 && zero <= k0 + 1) return;
    const int b = (int)blockIdx.x;
    if (b == 0) {
        panel<R, NB, MAXT, true>(S.p, W, L, L1, n, k0 + NB, nb, rowmap, rowmap1, pivots, moved, st);
    } else if (b == 1) {
        if (threadIdx.x < 64) det_accumulate<NB>(pivots, moved, k0, NB, st);
    } else {
        trail<NB, TR, MAXT / 64>(S.t, W, L, n, k0, k0 + NB + (b - 2) / ncb * ((int)blockDim.x / 64 * TR),
                                 k0 + 2 * NB + (b - 2) % ncb * 64, rowmap);
    }
}

// Panels with as few rows per thread as 512 threads allow: two waves per SIMD cover each other's
// latencies (a panel of 16 columns and 512-1000 rows takes 24 us so, 29 with four rows in each of
// 256 threads, 37 and more with a row in each of 1024).  Narrower panels only where the rows need
// 1024 threads.
hipError_t launch_panels(double* W, double* L, int n, int32_t* rowmap, double* pivots, int32_t* moved, DetState* st,
                         hipStream_t s) {
    constexpr int NB = GPANEL;
    int k0 = 0;
    for (; n - k0 > 2048; k0 += 8) {  // rows that need 1024 threads: 8 columns, panel and update in turn
        const int rows = n - k0, m = rows - 8;
        hipLaunchKernelGGL((g_panel<4, 8, 1024>), dim3(1), dim3((unsigned)(((rows + 3) / 4 + 63) / 64 * 64)), 0, s, W, L, n, k0, 8,
                           rowmap, pivots, moved, st);
        hipLaunchKernelGGL((g_trail<8, 4>), dim3((m + 63) / 64, (m + 15) / 16 + 1), dim3(256), 0, s, W, L, n, k0, rowmap,
                           pivots, moved, st);
    }
    double* Lx[2] = {L, L + (int64_t)NB * n};
    int32_t* rx[2] = {rowmap, rowmap + n};
    auto threads = [](int rows) {
        const int per = rows <= 512 ? 1 : rows <= 1024 ? 2 : 4;
        return dim3((unsigned)(((rows + per - 1) / per + 63) / 64 * 64));
    };
    {
        const int rows = n - k0, nb = std::min(rows, NB);
#define SGG_PANEL(R) hipLaunchKernelGGL((g_panel<R, NB, 512>), dim3(1), threads(rows), 0, s, W, Lx[0], n, k0, nb, rx[0], pivots, moved, st)
        if (rows <= 512) SGG_PANEL(1);
        else if (rows <= 1024) SGG_PANEL(2);
        else SGG_PANEL(4);
#undef SGG_PANEL
    }
    int cur = 0;
    for (; n - k0 > NB; k0 += NB, cur ^= 1) {
        const int rows = n - k0 - NB, nb = std::min(rows, NB), behind = rows - NB;
        const dim3 t = threads(rows);
        const int per = (int)t.x / 64 * 4, ncb = std::max(1, (behind + 63) / 64);
        const int blocks = 2 + (behind > 0 ? ncb * ((rows + per - 1) / per) : 0);
#define SGG_STEPS(R) hipLaunchKernelGGL((g_step<R, NB, 512, 4>), dim3(blocks), t, 0, s, W, Lx[cur], Lx[cur ^ 1], n, k0, nb, ncb, \
                                        rx[cur], rx[cur ^ 1], pivots, moved, st)
        if (rows <= 512) SGG_STEPS(1);
        else if (rows <= 1024) SGG_STEPS(2);
        else SGG_STEPS(4);
#undef SGG_STEPS
    }
    hipLaunchKernelGGL((g_product<NB>), dim3(1), dim3(64), 0, s, pivots, moved, k0, n - k0, st);
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
        c->w = dev_alloc(ctx, (size_t)std::max<int64_t>(n * n, 1) * 8 + 512 + (size_t)std::min<int64_t>(n, GPANEL_MAX) * (20 + 2 * GPANEL * 8));
        if (!c->w) return fail(ctx, SG_E_OOM, "determinant: workspace");
        c->n = n;
    }
    double* W = (double*)c->w;
    DetState* st = (DetState*)((char*)c->w + (((size_t)std::max<int64_t>(n * n, 1) * 8 + 255) & ~(size_t)255));
    // by panels, behind the state: the multipliers of two panels, the pivots, the row positions
    // after each of the two, exchange flags
    const bool panels = n > 0 && n <= GPANEL_MAX;
    double* L = (double*)((char*)st + 256);
    double* pivots = L + 2 * GPANEL * n;
    int32_t* rowmap = (int32_t*)(pivots + n);
    int32_t* moved = rowmap + 2 * n;
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
