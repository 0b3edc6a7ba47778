#pragma once
// Lean streaming pass: the interpreter for programs that keep one running value.
//
// A lean program reads at most two inputs into two registers; every value operation, predicate
// and reduction works in place on register 0 (a zip's second operand is register 1), nothing is
// compacted, and there is no exp, division, constant or move (lean_program decides).  Most
// chains, and every contract over a computed collection, have this form.  The general
// interpreter is bound by issue on them: 32 register moves around the 32 instructions of an
// affine (operands copied in and out of a five-register file), per-element bit fields for
// checks that hold, a wait for the neighbour load of a sortedness check in every sub-tile, and
// two waves per SIMD at 190-246 VGPRs.  Here no register index is dynamic, a check of a class
// or range test takes about one instruction per element, and four waves per SIMD hide each
// other's loads and dispatch, so nothing is prefetched.
//
// One sorted / all-finite check over 10^8 floats: 106 us (3.8 TB/s), before 202 / 172; the 2^20
// chain with three clauses: 14 us, before 56; 256 chains of 2^10 .. 2^22 elements (786 MB) in
// one batch at 256 x 4, 4 sub-tiles: 258 us (3.0 TB/s), before 535.  Bound by issue: with a
// quarter of the elements per lane (unroll 1) the dispatch doubles the batch's time.
//
// Layout, accumulation order, publication and finalization are the streaming kernel's, so a
// launch of the same shape gives the same bits.
#include "sg_stream_kernel.h"

namespace sg {

struct LeanLds {
    static constexpr int kSums = LEAN_SUMS;
    uint64_t slot[LEAN_BLOCK / 64][MAX_SLOTS];
    double sum[LEAN_BLOCK / 64][LEAN_SUMS];
    double tsum[TILE_BUF][LEAN_SUMS];
    int64_t tile[TILE_BUF];
    double fin[LEAN_BLOCK / 64][LEAN_SUMS];
};

// Dynamic LDS: [lds_slots][blockDim] u64, each lane's exact accumulators.
template <int U, bool INLINE>
__global__ __launch_bounds__(LEAN_BLOCK, 4) void lean_kernel(const StreamArgs A) {
    constexpr int V = 4 * U;
    constexpr int RW = 256 * U;  // elements of a wave's part of a sub-tile
    __shared__ LeanLds L;
    extern __shared__ uint64_t lacc[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int B = blockDim.x, nwaves = B >> 6, C = A.substeps;
    const int SUB = B * V;  // elements of a sub-tile
    const uint32_t epoch = A.epoch_ptr
        ? __builtin_amdgcn_readfirstlane(__hip_atomic_load(A.epoch_ptr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
        : A.epoch_val;
    const uint32_t wraw = A.limit_ptr
        ? __builtin_amdgcn_readfirstlane(__hip_atomic_load(A.limit_ptr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
        : A.wait_limit;
    const uint32_t wlimit = wraw == 0 ? kDefaultWaitSpins : wraw - 1u;
    const kptr kargs = (kptr)__builtin_amdgcn_kernarg_segment_ptr();
    const kptr kdesc = kargs + __builtin_offsetof(StreamArgs, inst0);
    const kptr kprog = kargs + __builtin_offsetof(StreamArgs, prog0);

    double rsum0 = 0.0, rsum1 = 0.0;  // the lane's float64 sums
    for (int k = 0; k < A.lds_slots; ++k) lacc[k * B + tid] = 0;  // a lane reads only its own
    auto acc_add = [&](int k, uint64_t v) { lacc[k * B + tid] += v; };
    auto acc_max = [&](int k, uint64_t v) {
        const uint64_t o = lacc[k * B + tid];
        lacc[k * B + tid] = v > o ? v : o;
    };
    auto acc_take = [&](int k) -> uint64_t {
        const uint64_t v = lacc[k * B + tid];
        lacc[k * B + tid] = 0;
        return v;
    };
    auto sum_add = [&](int k, double v) {
        if (k == 0) rsum0 += v;
        else rsum1 += v;
    };
    auto sum_take = [&](int k) -> double {
        double v;
        if (k == 0) { v = rsum0; rsum0 = 0.0; }
        else { v = rsum1; rsum1 = 0.0; }
        return v;
    };

    int cur = -1, ntl = 0;
    const char* D = nullptr;     // batched: descriptor in global memory
    const char* prog = nullptr;  // batched: program in global memory
    int plen = 0, nin = 0, flags = 0, nsum = 0, ns = 0;
    int64_t n = 0, tile0 = 0, ntiles = 0;
    const gu32 *in0 = nullptr, *in1 = nullptr;
    auto flush = [&]() {
        flush_instance<INLINE>(A, L, kdesc, D, cur, tile0, ntiles, ns, nsum, ntl, epoch, wlimit, acc_take, sum_take);
    };
    // one 16-byte scalar load per operation
    auto op_at = [&](int pc) -> SgOp {
        typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
        const int off = pc * (int)sizeof(SgOp);
        const u32x4 w = INLINE ? *(const SG_AS4 u32x4*)(kprog + off) : *(const SG_AS4 u32x4*)(const SG_AS4 char*)(prog + off);
        SgOp op;
        uint32_t* ow = (uint32_t*)&op;
        ow[0] = w.x; ow[1] = w.y; ow[2] = w.z; ow[3] = w.w;
        return op;
    };

    for (int64_t t = blockIdx.x; t < A.total_tiles; t += gridDim.x) {
        const int inst = INLINE ? 0 : (int)uload32(A.tile_inst + t);
        if (inst != cur || ntl == TILE_BUF) {
            if (cur >= 0) flush();
            if (inst != cur) {
                cur = inst;
                D = INLINE ? nullptr : (const char*)(A.insts + inst);
#define SG_D32(F) d32<INLINE>(kdesc, D, (int)__builtin_offsetof(InstDesc, F))
#define SG_D64(F) d64<INLINE>(kdesc, D, (int)__builtin_offsetof(InstDesc, F))
                prog = INLINE ? nullptr : (const char*)(A.progs + (int)SG_D32(prog_off));
                plen = (int)SG_D32(prog_len);
                const int64_t* n_dev = (const int64_t*)(uintptr_t)SG_D64(n_dev);
                n = n_dev ? (int64_t)uload64(n_dev) : (int64_t)SG_D64(n);
                if (INLINE && A.skip && uload64(A.skip) == 0) n = 0;
                tile0 = (int64_t)SG_D64(tile0);
                ntiles = (int64_t)SG_D64(ntiles);
                nin = (int)SG_D32(nin);
                flags = (int)SG_D32(flags);
                nsum = (int)SG_D32(nsum);
                ns = (int)SG_D32(nslots);
                in0 = gin(SG_D64(in[0]));
                in1 = gin(SG_D64(in[1]));
#undef SG_D32
#undef SG_D64
            }
        }
        const int64_t tbase = (t - tile0) * C * SUB;
        for (int c = 0; c < C; ++c) {
            const int64_t base = tbase + (int64_t)c * SUB;
            // elements left in the vector, as far as this sub-tile can tell (one past its end)
            const int64_t left = n - base;
            if (left <= 0) break;
            const int rem = left > SUB ? SUB + 1 : (int)left;
            const bool full = rem >= SUB;
            const bool vec = full && (flags & 1);
            int el = wave * RW + lane * 4;  // the lane's first element in the sub-tile
            uint32_t R0[V], R1[V];
            if (vec) {
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const sg_u32x4 w = *(const gu4*)(in0 + base + (el + u * 256));
                    R0[4 * u + 0] = w.x; R0[4 * u + 1] = w.y; R0[4 * u + 2] = w.z; R0[4 * u + 3] = w.w;
                }
                if (nin > 1) {
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        const sg_u32x4 w = *(const gu4*)(in1 + base + (el + u * 256));
                        R1[4 * u + 0] = w.x; R1[4 * u + 1] = w.y; R1[4 * u + 2] = w.z; R1[4 * u + 3] = w.w;
                    }
                }
            } else {
#pragma unroll
                for (int v = 0; v < V; ++v) {
                    const int i = el + (v >> 2) * 256 + (v & 3);
                    R0[v] = i < rem && i < SUB ? in0[base + i] : 0u;
                }
                if (nin > 1) {
#pragma unroll
                    for (int v = 0; v < V; ++v) {
                        const int i = el + (v >> 2) * 256 + (v & 3);
                        R1[v] = i < rem && i < SUB ? in1[base + i] : 0u;
                    }
                }
            }
            // first element after the wave's part (a sortedness check's last neighbour)
            uint32_t nbr = 0u;
            if (flags & 2) {
                const int ex = (wave + 1) * RW;
                if (ex < rem) nbr = in0[base + ex];
            }
            uint32_t S[MAX_SPACES];
            uint32_t P0 = 0, P1 = 0, P2 = 0, P3 = 0;
            S[0] = all_bits<V>();
            if (!full) {
                S[0] = 0;
#pragma unroll
                for (int v = 0; v < V; ++v) S[0] |= (el + (v >> 2) * 256 + (v & 3) < rem ? 1u : 0u) << v;
            }
            // index of a bit field's first element, in the accumulators' encoding
            auto first_of = [&](uint32_t m) -> uint64_t {
                const int v = __builtin_ctz(m);
                return ~(uint64_t)(base + el + (v >> 2) * 256 + (v & 3));
            };
            auto push = [&](uint32_t bits) { P3 = P2; P2 = P1; P1 = P0; P0 = bits; };
            auto pop = [&]() { P0 = P1; P1 = P2; P2 = P3; };
#define SG_EACH(...) _Pragma("unroll") for (int v = 0; v < V; ++v) { __VA_ARGS__ }
#define SG_MAP_F(CODE, EXPR) case CODE: { const float c0 = op.c0.f, c1 = op.c1.f; (void)c0; (void)c1; \
                SG_EACH(const float a = uf(R0[v]); R0[v] = fu(EXPR);) } break;
#define SG_MAP_I(CODE, EXPR) case CODE: { const uint32_t c0 = (uint32_t)op.c0.i, c1 = (uint32_t)op.c1.i; (void)c0; (void)c1; \
                SG_EACH(const uint32_t a = R0[v]; R0[v] = (EXPR);) } break;
#define SG_ZIP(CODE, EXPR) case CODE: { SG_EACH(const uint32_t a = R0[v], b = R1[v]; R0[v] = (EXPR);) } break;
#define SG_TEST(COND) { uint32_t bits = 0; SG_EACH(const uint32_t a = R0[v]; bits |= ((COND) ? 1u : 0u) << v;) push(bits); }
            SgOp op = op_at(0);
            for (int pc = 0; pc < plen; ++pc) {
                const SgOp next = op_at(pc + 1 < plen ? pc + 1 : pc);  // in flight while this one runs
                switch (op.code) {
                    SG_MAP_F(F_AFFINE, (a * c0) + c1)
                    SG_MAP_F(F_ADDC, a + c0)
                    SG_MAP_F(F_MULC, a * c0)
                    SG_MAP_F(F_SQUARE, a * a)
                    SG_MAP_F(F_NEG, -a)
                    SG_MAP_F(F_ABS, __builtin_fabsf(a))
                    SG_MAP_F(F_SQRT, __builtin_sqrtf(a))
                    SG_MAP_F(F_SQRT_ABS, __builtin_sqrtf(__builtin_fabsf(a)))
                    SG_MAP_I(I_AFFINE, a * c0 + c1)
                    SG_MAP_I(I_ADDC, a + c0)
                    SG_MAP_I(I_MULC, a * c0)
                    SG_MAP_I(I_SQUARE, a * a)
                    SG_MAP_I(I_NEG, 0u - a)
                    SG_MAP_I(I_ABS, ui(a) < 0 ? 0u - a : a)
                    SG_MAP_I(I_TO_F, fu((float)ui(a)))
                    SG_ZIP(F_ADD, fu(uf(a) + uf(b)))
                    SG_ZIP(F_SUB, fu(uf(a) - uf(b)))
                    SG_ZIP(F_MUL, fu(uf(a) * uf(b)))
                    SG_ZIP(I_ADD, a + b)
                    SG_ZIP(I_SUB, a - b)
                    SG_ZIP(I_MUL, a * b)
                    case P_CMP_F: {
                        const float k = op.c0.f;
                        switch (op.aux) {
                            case CMP_LT: SG_TEST(uf(a) < k) break;
                            case CMP_LE: SG_TEST(uf(a) <= k) break;
                            case CMP_GT: SG_TEST(uf(a) > k) break;
                            case CMP_GE: SG_TEST(uf(a) >= k) break;
                            case CMP_EQ: SG_TEST(uf(a) == k) break;
                            default: SG_TEST(uf(a) != k) break;
                        }
                    } break;
                    case P_CMP_I: {
                        const int32_t k = op.c0.i;
                        switch (op.aux) {
                            case CMP_LT: SG_TEST(ui(a) < k) break;
                            case CMP_LE: SG_TEST(ui(a) <= k) break;
                            case CMP_GT: SG_TEST(ui(a) > k) break;
                            case CMP_GE: SG_TEST(ui(a) >= k) break;
                            case CMP_EQ: SG_TEST(ui(a) == k) break;
                            default: SG_TEST(ui(a) != k) break;
                        }
                    } break;
                    case P_FINITE: SG_TEST(!__builtin_amdgcn_class(uf(a), 0x1 | 0x2 | 0x4 | 0x200)) break;
                    case P_RANGE_F: SG_TEST(uf(a) >= op.c0.f && uf(a) <= op.c1.f) break;
                    case P_RANGE_I: SG_TEST(ui(a) >= op.c0.i && ui(a) <= op.c1.i) break;
                    case P_TRUE: push(all_bits<V>()); break;
                    case P_AND: { const uint32_t b = P0 & P1; P0 = b; P1 = P2; P2 = P3; } break;
                    case P_OR: { const uint32_t b = P0 | P1; P0 = b; P1 = P2; P2 = P3; } break;
                    case P_NOT: P0 = ~P0 & all_bits<V>(); break;
                    case FILTER: {
                        const uint32_t m = get_space(S, op.sp2) & P0;
                        set_space(S, op.sp, m);
                        pop();
                    } break;
                    case CHK_ALL: case CHK_ANY: {
                        const uint32_t m = get_space(S, op.sp);
                        const uint32_t hit = op.code == CHK_ALL ? (m & ~P0) : (m & P0);
                        pop();
                        if (hit) acc_max(op.aux, first_of(hit));
                    } break;
                    case CHK_PRED: {
                        // for_all of a class or range test.  Where every element of the sub-tile is
                        // in the space, the lane's extrema decide it (three-operand instructions,
                        // about one per element; the float ones propagate NaN, which no bound
                        // admits); per-element bits are formed only when an element fails, in a
                        // filtered space or in the last sub-tile.
                        const uint8_t pc_ = op.pad;
                        bool bits = !(op.sp == 0 && full);
                        auto quick = [&](const uint32_t(&r)[V]) {
                            if (pc_ == P_FINITE) {
                                // not finite: the bits reach 0x7F800000 as a signed integer (+inf,
                                // positive NaNs) or 0xFF800000 as an unsigned one (-inf, negative NaNs)
                                int32_t ms = INT32_MIN;
                                uint32_t mu = 0u;
                                SG_EACH(ms = max(ms, ui(r[v])); mu = max(mu, r[v]);)
                                bits = (__ballot(ms >= 0x7F800000) | __ballot(mu >= 0xFF800000u)) != 0;
                            } else if (pc_ == P_RANGE_F) {
                                float hi = uf(0xFF800000u), lo = uf(0x7F800000u);
                                SG_EACH(hi = __builtin_elementwise_maximum(hi, uf(r[v]));
                                        lo = __builtin_elementwise_minimum(lo, uf(r[v]));)
                                bits = (__ballot(!(lo >= op.c0.f)) | __ballot(!(hi <= op.c1.f))) != 0;
                            } else {
                                int32_t hi = INT32_MIN, lo = INT32_MAX;
                                SG_EACH(hi = max(hi, ui(r[v])); lo = min(lo, ui(r[v]));)
                                bits = (__ballot(lo < op.c0.i) | __ballot(hi > op.c1.i)) != 0;
                            }
                        };
                        if (!bits) {
                            if (op.a == 0) quick(R0);
                            else quick(R1);
                        }
                        if (bits) {
                            uint32_t ok = 0;
                            SG_EACH(const uint32_t a = op.a == 0 ? R0[v] : R1[v];
                                    const bool in_f = uf(a) >= op.c0.f && uf(a) <= op.c1.f;
                                    const bool in_i = ui(a) >= op.c0.i && ui(a) <= op.c1.i;
                                    const bool fin = !__builtin_amdgcn_class(uf(a), 0x1 | 0x2 | 0x4 | 0x200);
                                    ok |= ((pc_ == P_FINITE ? fin : pc_ == P_RANGE_F ? in_f : in_i) ? 1u : 0u) << v;)
                            const uint32_t hit = get_space(S, op.sp) & ~ok;
                            if (hit) acc_max(op.aux, first_of(hit));
                        }
                    } break;
                    case CHK_SORTED_F: case CHK_SORTED_I: {
                        // the next lane's first element comes by a data-parallel shift, the next
                        // chunk's from lane 0, the next part's was loaded with the sub-tile
                        auto sorted = [&](auto le) {
                            uint32_t nx[U];
                            uint64_t found = 0;
#pragma unroll
                            for (int u = 0; u < U; ++u) {
                                uint32_t nxt = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)R0[4 * u], 0x130, 0xF, 0xF, false);  // wave_shl:1
                                const uint32_t last = u + 1 < U ? (uint32_t)__builtin_amdgcn_readfirstlane((int)R0[4 * ((u + 1) % U)]) : nbr;
                                nx[u] = lane == 63 ? last : nxt;
#pragma unroll
                                for (int j = 0; j < 4; ++j)
                                    found |= __ballot(!le(R0[4 * u + j], j < 3 ? R0[4 * u + (j + 1) % 4] : nx[u]));
                            }
                            if (found == 0) return;
                            // elements with a successor in range: all but in the vector's last sub-tile
                            uint32_t bad = 0;
                            int e1 = el + 1;
                            asm volatile("" : "+v"(e1));  // the range tests are formed here, not hoisted
#pragma unroll
                            for (int v = 0; v < V; ++v) {
                                const uint32_t b = (v & 3) < 3 ? R0[(v & ~3) + ((v & 3) + 1) % 4] : nx[v >> 2];
                                bad |= (!le(R0[v], b) && e1 + (v >> 2) * 256 + (v & 3) < rem ? 1u : 0u) << v;
                            }
                            if (bad) acc_max(op.aux, first_of(bad));
                        };
                        if (op.code == CHK_SORTED_F) sorted([](uint32_t a, uint32_t b) { return uf(a) <= uf(b); });
                        else sorted([](uint32_t a, uint32_t b) { return ui(a) <= ui(b); });
                    } break;
                    case RED_SUM_F: case RED_ABSSUM_F: {
                        const uint32_t m = get_space(S, op.sp);
                        double acc = 0.0;
                        if (op.code == RED_SUM_F && op.sp == 0 && full) {
                            SG_EACH(acc += (double)uf(R0[v]);)
                        } else {
                            // an element outside the space adds +0.0 (its bits masked to zero)
                            const uint32_t abs = op.code == RED_ABSSUM_F ? 0x7FFFFFFFu : 0xFFFFFFFFu;
                            SG_EACH(acc += (double)uf(R0[v] & lane_mask_bit(m, v) & abs);)
                        }
                        sum_add(op.aux, acc);
                    } break;
                    case RED_SUM_I: {
                        const uint32_t m = get_space(S, op.sp);
                        int64_t acc = 0;
                        SG_EACH(acc += (int64_t)ui(R0[v] & lane_mask_bit(m, v));)
                        acc_add(op.aux, (uint64_t)acc);
                    } break;
                    case RED_MAX_F: case RED_MIN_F: {
                        // IEEE maximum / minimum (NaN when any operand is NaN, -0 below +0) of the
                        // lane's elements in the space, then one order-preserving key per lane
                        const uint32_t m = get_space(S, op.sp);
                        const bool is_max = op.code == RED_MAX_F;
                        float hi = uf(0xFF800000u), lo = uf(0x7F800000u);
                        if (is_max) {
                            SG_EACH(const uint32_t km = lane_mask_bit(m, v);
                                    hi = __builtin_elementwise_maximum(hi, uf((R0[v] & km) | (0xFF800000u & ~km)));)
                        } else {
                            SG_EACH(const uint32_t km = lane_mask_bit(m, v);
                                    lo = __builtin_elementwise_minimum(lo, uf((R0[v] & km) | (0x7F800000u & ~km)));)
                        }
                        const uint32_t u = fu(is_max ? hi : lo);
                        uint32_t e = u ^ ((uint32_t)((int32_t)u >> 31) | 0x80000000u);
                        if (!is_max) e = ~e;
                        e = (u & 0x7FFFFFFFu) > 0x7F800000u ? 0xFFFFFFFFu : e;
                        acc_max(op.aux, (uint64_t)(m ? e : 0u));  // a lane with no element adds nothing
                    } break;
                    case RED_MAX_I: case RED_MIN_I: {
                        const uint32_t m = get_space(S, op.sp);
                        const bool is_max = op.code == RED_MAX_I;
                        int32_t hi = INT32_MIN, lo = INT32_MAX;
                        if (is_max) {
                            SG_EACH(const uint32_t km = lane_mask_bit(m, v); hi = max(hi, ui((R0[v] & km) | (0x80000000u & ~km)));)
                        } else {
                            SG_EACH(const uint32_t km = lane_mask_bit(m, v); lo = min(lo, ui((R0[v] & km) | (0x7FFFFFFFu & ~km)));)
                        }
                        uint32_t e = (uint32_t)(is_max ? hi : lo) ^ 0x80000000u;
                        if (!is_max) e = ~e;
                        acc_max(op.aux, (uint64_t)(m ? e : 0u));
                    } break;
                    case RED_COUNT: acc_add(op.aux, (uint64_t)__builtin_popcount(get_space(S, op.sp))); break;
                    case EMIT: {
                        gu32* q = gout(d64<INLINE>(kdesc, D, (int)__builtin_offsetof(InstDesc, out) + 8 * op.aux));
                        if (vec) {
#pragma unroll
                            for (int u = 0; u < U; ++u) {
                                sg_u32x4 w;
                                w.x = R0[4 * u + 0]; w.y = R0[4 * u + 1]; w.z = R0[4 * u + 2]; w.w = R0[4 * u + 3];
                                *(gu4*)(q + base + (el + u * 256)) = w;
                            }
                        } else {
                            uint32_t ib = S[0];
                            asm volatile("" : "+v"(ib));  // the masks are formed here, not hoisted
                            SG_EACH(if ((ib >> v) & 1u) q[base + (el + (v >> 2) * 256 + (v & 3))] = R0[v];)
                        }
                    } break;
                    default: break;
                }
                op = next;
            }
#undef SG_EACH
#undef SG_MAP_F
#undef SG_MAP_I
#undef SG_ZIP
#undef SG_TEST
        }
        // batched launch, tile end: its sums, over the lanes and then the waves in a fixed order,
        // are buffered for publication (a single program keeps per-lane sums until it flushes)
        if (!INLINE) {
            for (int k = 0; k < nsum; ++k) {
                const double s = wave_sum_f64(sum_take(k));
                if (lane == 0) L.sum[wave][k] = s;
            }
            lds_barrier();
            if (tid < nsum) {
                double s = 0.0;
                for (int w = 0; w < nwaves; ++w) s += L.sum[w][tid];
                L.tsum[ntl][tid] = s;
            }
            if (tid == 0) L.tile[ntl] = t;
            lds_barrier();
        }
        ntl = INLINE ? 1 : ntl + 1;
    }
    if (cur >= 0) flush();
    // the finalizing block has seen every block's words, so all of them have read the word
    if (INLINE && A.skip && tid == 0 && (int64_t)blockIdx.x == (ntiles - 1) % (int64_t)gridDim.x) st_relaxed(A.skip, 0);
}

}  // namespace sg
