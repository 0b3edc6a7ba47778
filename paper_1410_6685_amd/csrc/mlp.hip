// Cost model of the plan selector: a 24-64-64-1 float32 MLP with ReLU, trained on measured
// plan timings (mean squared error, Adam after Kingma and Ba, ICLR 2015) and evaluated for
// every candidate plan of a chain.
//
// A training step is forward, backward and update of a batch of at most 128 samples, its
// phases separated by barriers.  Every activation and every gradient is one thread's sum in a
// fixed order (inputs, units or samples ascending, product and sum rounded separately), so the
// results do not depend on how the work is divided and are identical from run to run.
// Inference runs one sample per thread over a grid.
//
// Parameter layout (floats): W1[24][64] | b1[64] | W2[64][64] | b2[64] | W3[64] | b3.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <cstring>
#include <string>
#include <vector>

#include "sg_runtime.h"

namespace sg {

constexpr int MI = 24, MH = 64, MB = 128;
constexpr int OW1 = 0, OB1 = OW1 + MI * MH, OW2 = OB1 + MH, OB2 = OW2 + MH * MH, OW3 = OB2 + MH, OB3 = OW3 + MH;
constexpr int MP = OB3 + 1;  // 5825
constexpr int HP = MH + 1;   // padded activation row (no LDS bank conflicts)

struct MlpLds {
    float w[MP];
    float x[MB][MI + 1];
    float h1[MB][HP];
    float h2[MB][HP];   // reused for dH1 after the output layer's gradient
    float d2[MB][HP];
    float dy[MB];
    float loss[MB];
};

struct AdamArgs {
    float lr, b1, b2, eps;
};

// Gradient and loss of one batch in one workgroup: the network and the batch's activations fit
// in LDS.  A thread per sample and unit (a call with 128 samples 217 -> 173 us, with one 182 -> 62,
// against a thread per sample).
static_assert(256 % MH == 0, "a thread keeps its unit from sample to sample");
__global__ __launch_bounds__(256) void mlp_grad_kernel(const float* __restrict__ P, float* __restrict__ G,
                                                      const float* __restrict__ X, const float* __restrict__ T, int B,
                                                      double* loss_out) {
    extern __shared__ char smem[];
    MlpLds& L = *reinterpret_cast<MlpLds*>(smem);
    const int tid = threadIdx.x, nt = blockDim.x;
    for (int i = tid; i < MP; i += nt) L.w[i] = P[i];
    for (int i = tid; i < B * MI; i += nt) L.x[i / MI][i % MI] = X[i];
    __syncthreads();
    // a thread per sample and unit, each sum in its own order of terms
    for (int k = tid; k < B * MH; k += nt) {
        const int s = k / MH, j = k % MH;
        float a = L.w[OB1 + j];
        for (int i = 0; i < MI; ++i) a += L.x[s][i] * L.w[OW1 + i * MH + j];
        L.h1[s][j] = a > 0.f ? a : 0.f;
    }
    __syncthreads();
    for (int k = tid; k < B * MH; k += nt) {
        const int s = k / MH, j = k % MH;
        float a = L.w[OB2 + j];
        for (int i = 0; i < MH; ++i) a += L.h1[s][i] * L.w[OW2 + i * MH + j];
        L.h2[s][j] = a > 0.f ? a : 0.f;
    }
    __syncthreads();
    for (int s = tid; s < B; s += nt) {
        float y = L.w[OB3];
        for (int j = 0; j < MH; ++j) y += L.h2[s][j] * L.w[OW3 + j];
        const float e = y - T[s];
        L.loss[s] = e * e;
        L.dy[s] = 2.f * e / (float)B;
    }
    __syncthreads();
    for (int k = tid; k < B * MH; k += nt) {
        const int s = k / MH, j = k % MH;
        L.d2[s][j] = L.h2[s][j] > 0.f ? L.dy[s] * L.w[OW3 + j] : 0.f;
    }
    // output layer gradient (needs h2), then dH1 overwrites h2
    for (int j = tid; j < MH + 1; j += nt) {
        float g = 0.f;
        for (int s = 0; s < B; ++s) g += (j < MH ? L.h2[s][j] : 1.f) * L.dy[s];
        G[j < MH ? OW3 + j : OB3] = g;
    }
    __syncthreads();
    float w2[MH];  // row i of W2, the same for every sample of the thread (in LDS one bank holds the column)
#pragma unroll
    for (int j = 0; j < MH; ++j) w2[j] = P[OW2 + tid % MH * MH + j];
    for (int k = tid; k < B * MH; k += nt) {
        const int s = k / MH, i = k % MH;
        float a = 0.f;
#pragma unroll
        for (int j = 0; j < MH; ++j) a += L.d2[s][j] * w2[j];
        L.h2[s][i] = L.h1[s][i] > 0.f ? a : 0.f;  // dH1
    }
    __syncthreads();
    for (int k = tid; k < MH * MH + MH; k += nt) {
        float g = 0.f;
        if (k < MH * MH) {
            const int i = k / MH, j = k % MH;
            for (int s = 0; s < B; ++s) g += L.h1[s][i] * L.d2[s][j];
            G[OW2 + k] = g;
        } else {
            const int j = k - MH * MH;
            for (int s = 0; s < B; ++s) g += L.d2[s][j];
            G[OB2 + j] = g;
        }
    }
    for (int k = tid; k < MI * MH + MH; k += nt) {
        float g = 0.f;
        if (k < MI * MH) {
            const int i = k / MH, j = k % MH;
            for (int s = 0; s < B; ++s) g += L.x[s][i] * L.h2[s][j];
            G[OW1 + k] = g;
        } else {
            const int j = k - MI * MH;
            for (int s = 0; s < B; ++s) g += L.h2[s][j];
            G[OB1 + j] = g;
        }
    }
    if (tid == 0) {
        double l = 0.0;
        for (int s = 0; s < B; ++s) l += L.loss[s];
        *loss_out = l / B;
    }
}

// ---- training ------------------------------------------------------------------------------
//
// A step holds 3.9 M separately rounded products and sums: 26 us of one CU's vector units, and
// four times that when one thread takes a whole sample (239 us per step in one workgroup of 256
// threads).  16 workgroups share it.  Workgroup g runs the forward and backward of its share of
// the batch, a wave per sample and a lane per unit, with the network in LDS; the activations go
// through memory, and after a barrier of the workgroups each thread owns one parameter for the
// whole training: its gradient over the batch, its Adam moments in registers.  A second barrier
// publishes the parameters.  What workgroups exchange is stored and loaded past the XCDs' L2s
// (agent scope) instead of being released by an L2 write-back.  12.8 us per step of 128 samples
// (10,000 samples: 1.01 ms per epoch, before 18.9 ms), half of it the two barriers and the round
// trips that follow them.
constexpr int TG = 16, TT = 512;      // workgroups, threads of one
constexpr int TSW = MB / TG;          // samples of one: a wave each
constexpr int W2P = MH + 1;           // padded row of W2 in LDS (read along rows and columns)
constexpr int TI = MI / 4;            // input rows of a workgroup's block of W1
constexpr int TC = MH / 4;            // units of its blocks (4 x 4 blocks of W2 and W1)
static_assert(TT / 64 == TSW && TG == 16, "a wave per sample, 4 x 4 parameter blocks");

struct MlpShared {
    float h1[MB][MH], h2[MB][MH], d2[MB][MH], d1[MB][MH];
    float dy[MB], loss[MB];
    uint64_t arrived;  // workgroups that reached a barrier, over the whole launch; or GIVEN_UP
};
constexpr uint64_t GIVEN_UP = 1ull << 63;

__device__ __forceinline__ uint64_t xld(const void* p) {
    return __hip_atomic_load((const uint64_t*)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ float xldf(const float* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void xst(float* p, float v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// a + x[0] w[0] + x[1] w[WS] + ..., MH terms in order.  The LDS reads of 16 terms are issued together:
// left to itself the compiler may wait for each pair (its choice hangs on unrelated code; a step
// then takes 1.3 us more).
template <int WS>
__device__ __forceinline__ float dot_mh(float a, const float* x, const float* w) {
#pragma unroll 1
    for (int i = 0; i < MH; i += 16) {
        float xv[16], wv[16];
#pragma unroll
        for (int q = 0; q < 16; ++q) {
            xv[q] = x[i + q];
            wv[q] = w[(i + q) * WS];
        }
#pragma unroll
        for (int q = 0; q < 16; ++q) a += xv[q] * wv[q];
        __builtin_amdgcn_sched_group_barrier(0x100, 16, 0);  // the reads,
        __builtin_amdgcn_sched_group_barrier(0x002, 40, 0);  // then the arithmetic
    }
    return a;
}

// Train for `epochs` passes over n samples in batches of B (the last partial batch included).  The
// parameters at the start are kept behind P (the place of a gradient call's result).
__global__ __launch_bounds__(TT) void mlp_train_kernel(float* __restrict__ P, float* __restrict__ M1, float* __restrict__ M2,
                                                       const float* __restrict__ X, const float* __restrict__ T, int64_t n,
                                                       int B, int epochs, int step0, AdamArgs ad,
                                                       double* __restrict__ epoch_loss, MlpShared* ex, uint32_t limit) {
    __shared__ float w1[MI * MH], w2[MH * W2P], b1[MH], b2[MH], w3[MH], b3[1];
    __shared__ float sx[TSW][MI], sh1[TSW][MH], sh2[TSW][MH], sd2[TSW][MH];
    __shared__ float ch1[MB][TC], cd2[MB][TC], cd1[MB][TC], ch2[MB][TC], cx[MB][TI], cdy[MB], closs[MB], one[1];
    __shared__ int go;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int g = blockIdx.x, jb = g & 3, ib = g >> 2;
    // the parameter this thread owns (or -1), and the two columns whose products sum to its
    // gradient over the samples
    int own = -1;
    const float *pa = one, *pb = cdy;
    int sa = 0, sb = 1;
    if (tid < TC * TC) {
        const int i = tid / TC, j = tid % TC;
        own = OW2 + (ib * TC + i) * MH + jb * TC + j;
        pa = &ch1[0][i]; sa = TC;
        pb = &cd2[0][j]; sb = TC;
    } else if (tid < TC * TC + TI * TC) {
        const int i = (tid - TC * TC) / TC, j = tid % TC;
        own = OW1 + (ib * TI + i) * MH + jb * TC + j;
        pa = &cx[0][i]; sa = TI;
        pb = &cd1[0][j]; sb = TC;
    } else if (tid < TC * TC + TI * TC + TC) {
        const int j = tid % TC;
        if (ib == 0) { own = OB2 + jb * TC + j; pb = &cd2[0][j]; sb = TC; }
        else if (ib == 1) { own = OB1 + jb * TC + j; pb = &cd1[0][j]; sb = TC; }
        else if (ib == 2) { own = OW3 + jb * TC + j; pa = &ch2[0][j]; sa = TC; }
        else if (g == 3 * 4 && j == 0) own = OB3;
    }
    float p = 0.f, m1 = 0.f, m2 = 0.f;
    if (own >= 0) { p = P[own]; m1 = M1[own]; m2 = M2[own]; P[MP + own] = p; }
    if (tid == 0) one[0] = 1.f;
    uint64_t target = 0;
    // Every workgroup's stores so far are in memory before any workgroup passes.  The wait is bounded
    // (`limit` polls, seconds).  A workgroup gives up by marking the counter, and only while the
    // count is short, so the others read either the full count or the mark: all of them pass the
    // last barrier or none does.  Where none does, the host puts the parameters back (the moments
    // are written after the last barrier).
    auto barrier = [&]() -> bool {
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
        target += TG;
        if (tid == 0) {
            (void)__hip_atomic_fetch_add(&ex->arrived, (uint64_t)1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            // (v stays the same for the whole wave to the compiler: a scalar loop)
            uint64_t v = xld(&ex->arrived);
            for (uint32_t spins = 1; v < target && spins < limit; ++spins) v = xld(&ex->arrived);
            if (__builtin_expect(v < target, 0)) do {
                uint64_t seen = v;
                const bool marked = __hip_atomic_compare_exchange_strong(&ex->arrived, &seen, v | GIVEN_UP, __ATOMIC_RELAXED,
                                                                         __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                // (one that fails saw an arrival, of which there are at most TG)
                v = __builtin_amdgcn_readfirstlane(marked) ? GIVEN_UP : xld(&ex->arrived);
            } while (v < target);
            go = v < GIVEN_UP;
        }
        __syncthreads();
        return __builtin_amdgcn_readfirstlane(go) != 0;
    };
    int step = step0;
    for (int e = 0; e < epochs; ++e) {
        double tot = 0.0;
        int64_t cnt = 0;
        for (int64_t s0 = 0; s0 < n; s0 += B) {
            const int b = (int)(n - s0 < B ? n - s0 : B);
            ++step;
            // ---- this workgroup's samples: forward, then the gradients of the units ----
            {
                constexpr int NP = (MP - 1) / 2, Q = (NP + TT - 1) / TT;
                uint64_t v[Q];
#pragma unroll
                for (int q = 0; q < Q; ++q) v[q] = tid + q * TT < NP ? xld(P + 2 * (tid + q * TT)) : 0;
                const float last = tid == 0 ? xldf(P + MP - 1) : 0.f;
#pragma unroll
                for (int q = 0; q < Q; ++q) {
                    const int i = 2 * (tid + q * TT);
                    if (i >= 2 * NP) continue;
#pragma unroll
                    for (int h = 0; h < 2; ++h) {  // the arrays' bounds are even
                        const float f = __builtin_bit_cast(float, (uint32_t)(v[q] >> (32 * h)));
                        const int k = i + h;
                        if (k < OB1) w1[k - OW1] = f;
                        else if (k < OW2) b1[k - OB1] = f;
                        else if (k < OB2) w2[(k - OW2) / MH * W2P + (k - OW2) % MH] = f;
                        else if (k < OW3) b2[k - OB2] = f;
                        else w3[k - OW3] = f;
                    }
                }
                if (tid == 0) b3[0] = last;
            }
            const int per = (b + TG - 1) / TG, lo = g * per;
            const int mine = b - lo < per ? (b - lo > 0 ? b - lo : 0) : per;
            if (tid < mine * MI) (&sx[0][0])[tid] = X[(s0 + lo) * MI + tid];
            for (int i = tid; i < b * TI; i += TT) (&cx[0][0])[i] = X[(s0 + i / TI) * MI + ib * TI + i % TI];
            __syncthreads();
            if (wave < mine) {
                const int s = lo + wave, j = lane;
                float a = b1[j];
#pragma unroll
                for (int i = 0; i < MI; ++i) a += sx[wave][i] * w1[i * MH + j];
                const float h1 = a > 0.f ? a : 0.f;
                sh1[wave][j] = h1;
                __builtin_amdgcn_wave_barrier();  // one wave's LDS accesses keep their order
                a = dot_mh<W2P>(b2[j], sh1[wave], w2 + j);
                const float h2 = a > 0.f ? a : 0.f;
                sh2[wave][j] = h2 * w3[j];
                __builtin_amdgcn_wave_barrier();
                float y = b3[0];
#pragma unroll 16
                for (int i = 0; i < MH; ++i) y += sh2[wave][i];
                const float er = y - T[s0 + s];
                const float dy = 2.f * er / (float)b;
                const float d2 = h2 > 0.f ? dy * w3[j] : 0.f;
                sd2[wave][j] = d2;
                __builtin_amdgcn_wave_barrier();
                a = dot_mh<1>(0.f, sd2[wave], w2 + j * W2P);
                const float d1 = h1 > 0.f ? a : 0.f;
                xst(&ex->h1[s][j], h1);
                xst(&ex->h2[s][j], h2);
                xst(&ex->d2[s][j], d2);
                xst(&ex->d1[s][j], d1);
                if (lane == 0) {
                    xst(&ex->dy[s], dy);
                    xst(&ex->loss[s], er * er);
                }
            }
            if (!barrier()) return;
            // ---- this workgroup's parameters: gradient over the batch, update ----
            for (int i = tid; i < b * (TC / 2); i += TT) {
                const int s = i / (TC / 2), c = 2 * (i % (TC / 2));
                const uint64_t x1 = xld(&ex->h1[s][ib * TC + c]), x2 = xld(&ex->d2[s][jb * TC + c]),
                               x3 = xld(&ex->d1[s][jb * TC + c]), x4 = ib == 2 ? xld(&ex->h2[s][jb * TC + c]) : 0;
                *(uint64_t*)&ch1[s][c] = x1;
                *(uint64_t*)&cd2[s][c] = x2;
                *(uint64_t*)&cd1[s][c] = x3;
                if (ib == 2) *(uint64_t*)&ch2[s][c] = x4;
            }
            if (tid < b) {
                cdy[tid] = xldf(&ex->dy[tid]);
                if (g == 0) closs[tid] = xldf(&ex->loss[tid]);
            }
            __syncthreads();
            if (own >= 0) {
                float gr = 0.f;
#pragma unroll 8
                for (int s = 0; s < b; ++s) gr += pa[s * sa] * pb[s * sb];
                const float c1 = 1.f - powf(ad.b1, (float)step), c2 = 1.f - powf(ad.b2, (float)step);
                m1 = ad.b1 * m1 + (1.f - ad.b1) * gr;
                m2 = ad.b2 * m2 + (1.f - ad.b2) * (gr * gr);
                p = p - ad.lr * (m1 / c1) / (sqrtf(m2 / c2) + ad.eps);
                xst(&P[own], p);
            } else if (g == 0 && tid == TT - 1) {
                double l = 0.0;
                for (int s = 0; s < b; ++s) l += closs[s];
                tot += l / b * b;
                cnt += b;
            }
            if (!barrier()) return;
        }
        if (g == 0 && tid == TT - 1) epoch_loss[e] = tot / (double)(cnt ? cnt : 1);
    }
    if (own >= 0) {
        M1[own] = m1;
        M2[own] = m2;
    }
}

__global__ __launch_bounds__(256) void mlp_predict_kernel(const float* __restrict__ P, const float* __restrict__ X,
                                                         int64_t n, float* __restrict__ Y) {
    __shared__ float w[MP];
    for (int i = threadIdx.x; i < MP; i += blockDim.x) w[i] = P[i];
    __syncthreads();
    const int64_t s = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (s >= n) return;
    float x[MI], h1[MH];
    for (int i = 0; i < MI; ++i) x[i] = X[s * MI + i];
    for (int j = 0; j < MH; ++j) {
        float a = w[OB1 + j];
        for (int i = 0; i < MI; ++i) a += x[i] * w[OW1 + i * MH + j];
        h1[j] = a > 0.f ? a : 0.f;
    }
    float y = w[OB3];
    for (int j = 0; j < MH; ++j) {
        float a = w[OB2 + j];
        for (int i = 0; i < MH; ++i) a += h1[i] * w[OW2 + i * MH + j];
        y += (a > 0.f ? a : 0.f) * w[OW3 + j];
    }
    Y[s] = y;
}


// Training data of the cost model.  One block per feature column: the column's mean and
// population standard deviation (two passes, float64, each thread's strided partial sums
// added lanes-then-waves in a fixed order), minimum and maximum.  stats[k] = {mean, std, lo,
// hi} as doubles.
__global__ __launch_bounds__(256) void mlp_colstats_kernel(const float* __restrict__ X, int64_t n,
                                                           double* __restrict__ stats) {
    __shared__ double red[4];
    __shared__ float rmin[4], rmax[4];
    const int k = blockIdx.x, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    auto block_sum = [&](double v) -> double {
        for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
        if (lane == 0) red[wave] = v;
        __syncthreads();
        const double t = (red[0] + red[1]) + (red[2] + red[3]);
        __syncthreads();
        return t;
    };
    double s = 0.0;
    float lo = __builtin_inff(), hi = -__builtin_inff();
    for (int64_t i = threadIdx.x; i < n; i += 256) {
        const float x = X[i * MI + k];
        s += (double)x;
        lo = fminf(lo, x);
        hi = fmaxf(hi, x);
    }
    const double mean = block_sum(s) / (double)n;
    double q = 0.0;
    for (int64_t i = threadIdx.x; i < n; i += 256) {
        const double d = (double)X[i * MI + k] - mean;
        q += d * d;
    }
    const double var = block_sum(q) / (double)n;
    for (int o = 32; o > 0; o >>= 1) {
        lo = fminf(lo, __shfl_xor(lo, o));
        hi = fmaxf(hi, __shfl_xor(hi, o));
    }
    if (lane == 0) { rmin[wave] = lo; rmax[wave] = hi; }
    __syncthreads();
    if (threadIdx.x == 0) {
        stats[4 * k + 0] = mean;
        stats[4 * k + 1] = __builtin_sqrt(var);
        stats[4 * k + 2] = fminf(fminf(rmin[0], rmin[1]), fminf(rmin[2], rmin[3]));
        stats[4 * k + 3] = fmaxf(fmaxf(rmax[0], rmax[1]), fmaxf(rmax[2], rmax[3]));
    }
}

// Xn = (X - mean) / scale per feature (float32 operations), T = log(1000 ms) (microseconds,
// computed in float64 and rounded to float32).
__global__ __launch_bounds__(256) void mlp_standardize_kernel(const float* __restrict__ X, const double* __restrict__ ms,
                                                              int64_t n, const float* __restrict__ mean,
                                                              const float* __restrict__ scale, float* __restrict__ Xn,
                                                              float* __restrict__ T) {
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i < n * MI) {
        const int k = (int)(i % MI);
        Xn[i] = (X[i] - mean[k]) / scale[k];
    }
    if (ms && i < n) T[i] = (float)log(ms[i] * 1000.0);
}

}  // namespace sg

using namespace sgrt;


extern "C" {

sg_status sg_mlp_create(sg_ctx ctx, const float* params, int64_t nparams, sg_mlp* out) {
    if (!ctx || !out || !params || nparams != sg::MP) return fail(ctx, SG_E_INVALID, "mlp_create: need 5825 initial parameters");
    auto* m = new sg_mlp_s();
    m->ctx = ctx;
    ctx_retain(ctx);
    if (hipMalloc(&m->P, 4 * sg::MP * sizeof(float)) != hipSuccess || hipMalloc(&m->loss, 1024 * sizeof(double)) != hipSuccess ||
        hipMalloc(&m->shared, sizeof(sg::MlpShared)) != hipSuccess) {
        (void)sg_mlp_release(m);
        return fail(ctx, SG_E_OOM, "mlp_create: allocation");
    }
    hipError_t e = hipMemsetAsync(m->P, 0, 4 * sg::MP * sizeof(float), ctx->stream);
    if (e == hipSuccess) e = hipMemcpyAsync(m->P, params, sg::MP * sizeof(float), hipMemcpyHostToDevice, ctx->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(ctx->stream);
    if (e != hipSuccess) {
        (void)sg_mlp_release(m);
        return hip_fail(ctx, e, "mlp_create: upload");
    }
    *out = m;
    return SG_OK;
}

sg_status sg_mlp_release(sg_mlp m) {
    if (!m) return SG_E_INVALID;
    sg_ctx_s* ctx = m->ctx;
    (void)hipStreamSynchronize(ctx->stream);
    if (m->P) (void)hipFree(m->P);
    if (m->loss) (void)hipFree(m->loss);
    if (m->shared) (void)hipFree(m->shared);
    delete m;
    ctx_release(ctx);
    return SG_OK;
}

sg_status sg_mlp_get_params(sg_mlp m, float* params, int64_t nparams) {
    if (!m || !params || nparams != sg::MP) return fail(m ? m->ctx : nullptr, SG_E_INVALID, "mlp_get_params: bad buffer");
    SG_HIP(m->ctx, hipMemcpyAsync(params, m->P, sg::MP * sizeof(float), hipMemcpyDeviceToHost, m->ctx->stream));
    SG_HIP(m->ctx, hipStreamSynchronize(m->ctx->stream));
    return SG_OK;
}

// Loss and gradient of one batch (no update): X_dev is B x 24, T_dev B floats (device).
sg_status sg_mlp_grad(sg_mlp m, const float* X_dev, const float* T_dev, int32_t B, float* grad_host, double* loss) {
    if (!m || !X_dev || !T_dev || B < 1 || B > sg::MB || !grad_host) return fail(m ? m->ctx : nullptr, SG_E_INVALID, "mlp_grad: bad argument (1 <= B <= 128)");
    sg_ctx_s* ctx = m->ctx;
    if (sg_status st = check_device_range(ctx, X_dev, (size_t)B * sg::MI * 4, "mlp_grad X")) return st;
    if (sg_status st = check_device_range(ctx, T_dev, (size_t)B * 4, "mlp_grad T")) return st;
    SG_HIP(ctx, hipFuncSetAttribute((const void*)sg::mlp_grad_kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                                    (int)sizeof(sg::MlpLds)));
    hipLaunchKernelGGL(sg::mlp_grad_kernel, dim3(1), dim3(256), sizeof(sg::MlpLds), ctx->stream, m->P, m->P + sg::MP,
                       X_dev, T_dev, (int)B, m->loss);
    SG_HIP(ctx, hipGetLastError());
    SG_HIP(ctx, hipMemcpyAsync(grad_host, m->P + sg::MP, sg::MP * sizeof(float), hipMemcpyDeviceToHost, ctx->stream));
    double l = 0;
    SG_HIP(ctx, hipMemcpyAsync(&l, m->loss, sizeof(double), hipMemcpyDeviceToHost, ctx->stream));
    SG_HIP(ctx, hipStreamSynchronize(ctx->stream));
    if (loss) *loss = l;
    return SG_OK;
}

// Train on n samples (device X n x 24, T n) for `epochs` epochs in batches of `batch` (<= 128),
// in the given sample order.  epoch_loss (host, `epochs` doubles) receives the mean loss.
sg_status sg_mlp_train(sg_mlp m, const float* X_dev, const float* T_dev, int64_t n, int32_t batch, int32_t epochs,
                       float lr, double* epoch_loss) {
    if (!m || !X_dev || !T_dev || n < 1 || batch < 1 || batch > sg::MB || epochs < 1 || epochs > 1000)
        return fail(m ? m->ctx : nullptr, SG_E_INVALID, "mlp_train: bad argument");
    sg_ctx_s* ctx = m->ctx;
    if (sg_status st = check_device_range(ctx, X_dev, (size_t)n * sg::MI * 4, "mlp_train X")) return st;
    if (sg_status st = check_device_range(ctx, T_dev, (size_t)n * 4, "mlp_train T")) return st;
    sg::AdamArgs ad{lr, 0.9f, 0.999f, 1e-8f};
    const char* name = "mlp_train";
    auto* ex = (sg::MlpShared*)m->shared;
    const uint32_t limit = ctx->wait_limit ? ctx->wait_limit - 1u : sg::kDefaultWaitSpins;
    std::vector<double> el(epochs);
    // The training workgroups have to be on the device together.  While other work holds it their
    // wait can end, with the model as it was, and the training is launched again; with a limit set by
    // the caller the first such end is reported.
    uint64_t arrived = sg::GIVEN_UP;
    for (int tries = 0; arrived >= sg::GIVEN_UP && tries < (ctx->wait_limit ? 1 : 8); ++tries) {
        // (a limit of no polls: given up before the first barrier)
        SG_HIP(ctx, hipMemsetAsync(&ex->arrived, limit ? 0 : 0x80, sizeof(uint64_t), ctx->stream));
        hipEvent_t a = nullptr, b = nullptr;
        if (ctx->timing) {
            (void)hipEventCreate(&a);
            (void)hipEventCreate(&b);
            (void)hipEventRecord(a, ctx->stream);
        }
        hipLaunchKernelGGL(sg::mlp_train_kernel, dim3(sg::TG), dim3(sg::TT), 0, ctx->stream, m->P, m->P + 2 * sg::MP,
                           m->P + 3 * sg::MP, X_dev, T_dev, n, (int)batch, (int)epochs, m->step, ad, m->loss, ex, limit);
        SG_HIP(ctx, hipGetLastError());
        if (ctx->timing) (void)hipEventRecord(b, ctx->stream);
        SG_HIP(ctx, hipMemcpyAsync(el.data(), m->loss, epochs * sizeof(double), hipMemcpyDeviceToHost, ctx->stream));
        SG_HIP(ctx, hipMemcpyAsync(&arrived, &ex->arrived, sizeof(arrived), hipMemcpyDeviceToHost, ctx->stream));
        SG_HIP(ctx, hipStreamSynchronize(ctx->stream));
        if (arrived >= sg::GIVEN_UP)
            SG_HIP(ctx, hipMemcpyAsync(m->P, m->P + sg::MP, sg::MP * sizeof(float), hipMemcpyDeviceToDevice, ctx->stream));
        if (ctx->timing) {
            float ms = 0.f;
            if (hipEventElapsedTime(&ms, a, b) == hipSuccess) { ctx->times[name].ms += ms; ctx->times[name].n += 1; }
            (void)hipEventDestroy(a);
            (void)hipEventDestroy(b);
        }
    }
    if (arrived >= sg::GIVEN_UP)
        return fail(ctx, SG_E_DEVICE, "mlp_train: a barrier of the training workgroups timed out; the model is unchanged");
    m->step += (int)(epochs * ((n + batch - 1) / batch));
    if (epoch_loss) std::memcpy(epoch_loss, el.data(), epochs * sizeof(double));
    return SG_OK;
}

// Predictions for n samples (device X n x 24 -> device Y n).
sg_status sg_mlp_predict(sg_mlp m, const float* X_dev, int64_t n, float* Y_dev) {
    if (!m || !X_dev || !Y_dev || n < 0) return fail(m ? m->ctx : nullptr, SG_E_INVALID, "mlp_predict: bad argument");
    if (n == 0) return SG_OK;
    sg_ctx_s* ctx = m->ctx;
    if (sg_status st = check_device_range(ctx, X_dev, (size_t)n * sg::MI * 4, "mlp_predict X")) return st;
    if (sg_status st = check_device_range(ctx, Y_dev, (size_t)n * 4, "mlp_predict Y")) return st;
    const unsigned grid = (unsigned)((n + 255) / 256);
    hipLaunchKernelGGL(sg::mlp_predict_kernel, dim3(grid), dim3(256), 0, ctx->stream, m->P, X_dev, n, Y_dev);
    SG_HIP(ctx, hipGetLastError());
    return SG_OK;
}

// Training data of the cost model, prepared on the device: fit the standardization on the
// raw features X (n x 24), then write the standardized features Xn and, when ms is given, the
// targets log(run time in microseconds).
sg_status sg_mlp_fit_data(sg_mlp m, const float* X_dev, const double* ms_dev, int64_t n, float* Xn_dev, float* T_dev) {
    if (!m || !X_dev || !Xn_dev || n < 1 || (ms_dev && !T_dev))
        return fail(m ? m->ctx : nullptr, SG_E_INVALID, "mlp_fit_data: bad argument");
    sg_ctx_s* ctx = m->ctx;
    if (sg_status st = check_device_range(ctx, X_dev, (size_t)n * sg::MI * 4, "mlp_fit_data X")) return st;
    if (sg_status st = check_device_range(ctx, Xn_dev, (size_t)n * sg::MI * 4, "mlp_fit_data Xn")) return st;
    if (ms_dev) {
        if (sg_status st = check_device_range(ctx, ms_dev, (size_t)n * 8, "mlp_fit_data ms")) return st;
        if (sg_status st = check_device_range(ctx, T_dev, (size_t)n * 4, "mlp_fit_data T")) return st;
    }
    // statistics (24 x 4 doubles), then the float32 mean and scale the kernels and the
    // selector use
    void* w = dev_alloc(ctx, sg::MI * 4 * sizeof(double) + 2 * sg::MI * sizeof(float));
    if (!w) return fail(ctx, SG_E_OOM, "mlp_fit_data: workspace");
    double* stats = (double*)w;
    float* msd = (float*)(stats + sg::MI * 4);
    double h[sg::MI * 4];
    hipLaunchKernelGGL(sg::mlp_colstats_kernel, dim3(sg::MI), dim3(256), 0, ctx->stream, X_dev, n, stats);
    hipError_t e = hipGetLastError();
    if (e == hipSuccess) e = hipMemcpyAsync(h, stats, sizeof(h), hipMemcpyDeviceToHost, ctx->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(ctx->stream);
    if (e != hipSuccess) {
        dev_free(ctx, w);
        return hip_fail(ctx, e, "mlp_fit_data: statistics");
    }
    float mean[sg::MI], scale[sg::MI], lo[sg::MI], hi[sg::MI], both[2 * sg::MI];
    for (int k = 0; k < sg::MI; ++k) {
        mean[k] = (float)h[4 * k];
        // a constant feature keeps scale 1 (it standardizes to 0)
        scale[k] = h[4 * k + 1] > 1e-6 ? (float)h[4 * k + 1] : 1.0f;
        lo[k] = (float)h[4 * k + 2];
        hi[k] = (float)h[4 * k + 3];
        both[k] = mean[k];
        both[sg::MI + k] = scale[k];
    }
    (void)sg_mlp_set_norm(m, mean, scale, lo, hi);
    e = hipMemcpyAsync(msd, both, sizeof(both), hipMemcpyHostToDevice, ctx->stream);
    if (e == hipSuccess) {
        const int64_t tot = n * sg::MI;
        hipLaunchKernelGGL(sg::mlp_standardize_kernel, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, ctx->stream,
                           X_dev, ms_dev, n, msd, msd + sg::MI, Xn_dev, T_dev);
        e = hipGetLastError();
    }
    if (e == hipSuccess) e = hipStreamSynchronize(ctx->stream);
    dev_free(ctx, w);
    if (e != hipSuccess) return hip_fail(ctx, e, "mlp_fit_data: standardize");
    return SG_OK;
}

// Standardized features of n samples with the model's fitted standardization (and targets).
sg_status sg_mlp_standardize(sg_mlp m, const float* X_dev, const double* ms_dev, int64_t n, float* Xn_dev, float* T_dev) {
    if (!m || !X_dev || !Xn_dev || n < 0 || (ms_dev && !T_dev))
        return fail(m ? m->ctx : nullptr, SG_E_INVALID, "mlp_standardize: bad argument");
    sg_ctx_s* ctx = m->ctx;
    if (!m->norm_set) return fail(ctx, SG_E_STATE, "mlp_standardize: the model has no standardization");
    if (n == 0) return SG_OK;
    if (sg_status st = check_device_range(ctx, X_dev, (size_t)n * sg::MI * 4, "mlp_standardize X")) return st;
    if (sg_status st = check_device_range(ctx, Xn_dev, (size_t)n * sg::MI * 4, "mlp_standardize Xn")) return st;
    if (ms_dev) {
        if (sg_status st = check_device_range(ctx, ms_dev, (size_t)n * 8, "mlp_standardize ms")) return st;
        if (sg_status st = check_device_range(ctx, T_dev, (size_t)n * 4, "mlp_standardize T")) return st;
    }
    float* msd = (float*)dev_alloc(ctx, 2 * sg::MI * sizeof(float));
    if (!msd) return fail(ctx, SG_E_OOM, "mlp_standardize: workspace");
    float both[2 * sg::MI];
    std::memcpy(both, m->mean, sizeof(m->mean));
    std::memcpy(both + sg::MI, m->scale, sizeof(m->scale));
    hipError_t e = hipMemcpyAsync(msd, both, sizeof(both), hipMemcpyHostToDevice, ctx->stream);
    if (e == hipSuccess) {
        const int64_t tot = n * sg::MI;
        hipLaunchKernelGGL(sg::mlp_standardize_kernel, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, ctx->stream,
                           X_dev, ms_dev, n, msd, msd + sg::MI, Xn_dev, T_dev);
        e = hipGetLastError();
    }
    if (e == hipSuccess) e = hipStreamSynchronize(ctx->stream);
    dev_free(ctx, msd);
    if (e != hipSuccess) return hip_fail(ctx, e, "mlp_standardize");
    return SG_OK;
}

}  // extern "C"
