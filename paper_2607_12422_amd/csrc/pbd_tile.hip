// Projection GEMM of passes with many rows (bf16 models; the same products and
// epilogues as pbd_gemm.hip): blocks of 4 to 12 x 8 to 16 tiles of 16 x 16 over
// the whole K, operands and weights shared through LDS.
//
// WM x WN computing waves own TM x TN tiles each; NL more waves copy the
// fragments of the block's next K steps (packed, 1 KiB each; KST steps a stage)
// straight into a ring of RING stages in LDS, so that the computing waves issue nothing but
// LDS reads and MFMAs.  One barrier per stage: the loaders wait for the stage's
// fragments before it, and fill the slot it releases after it.  A fragment
// comes to the CU once per block and to the registers once per wave row or
// column, TM + TN reads per TM * TN products: what a block of few tiles per
// wave spends on the path from the L2 (pbd_gemm.hip) goes to the matrix cores.
// Blocks this large leave the chip idle where a projection has few of them;
// gemm_pick (pbd_gemm.hip) chooses between the two.
#include "pbd_epi.h"
#include "pbd_launch.h"

#include <algorithm>

namespace pbd {
namespace {

template <bool PAIR, int WM, int WN, int TM, int TN, int NL, int KST, int RING> struct TL {
    static constexpr int XF = PAIR ? 2 : 1;
    static constexpr int BM = WM * TM, BN = WN * TN;           // tiles of a block
    static constexpr int NX = BM * XF + BN;                    // fragments of a K step
    static constexpr int PER = KST * NX / NL;                  // ... of a stage, per loader wave
    static constexpr int NC = WM * WN;                         // computing waves
    static constexpr size_t STAGE = (size_t)KST * NX * 1024, LDS = RING * STAGE;
    static_assert(KST * NX % NL == 0 && KST <= 2 && PER * (RING - 2) < 64 && RING >= 2 && RING <= 6, "loads in flight fit the wait counter");
};

template <bool PAIR, int WM, int WN, int TM, int TN, int NL, int KST, int RING, bool ARG>
__global__ __launch_bounds__((WM * WN + NL) * 64) __attribute__((amdgpu_waves_per_eu(3, 8))) void k_gemm_tile(BigGemmArgs a) {
    typedef TL<PAIR, WM, WN, TM, TN, NL, KST, RING> C;
    constexpr int ROWS = C::BM * 16, NSL = C::NC * WAVE / ROWS;
    static_assert(NSL >= 1, "a thread per row");
    const int lane = threadIdx.x % WAVE;
    const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE);
    const int lrow = lane % 16, lgrp = lane / 16;
    int bm, bn;
    if (!block_of(a, bm, bn)) return;
    const int mt0 = bm * C::BM, nt0 = bn * C::BN, kb = a.kb, n_st = kb / KST;   // kb is even
    extern __shared__ __align__(16) unsigned char ring[];
    __shared__ float s_part[NSL][ROWS];
    __shared__ float s_am[ARG ? WN : 1][3][ARG ? ROWS : 1];
    __shared__ int s_ai[ARG ? WN : 1][ARG ? ROWS : 1];

    if (wid >= C::NC) {
        typedef __attribute__((address_space(3))) void* lds;
        const int lw = wid - C::NC;
        const unsigned loff = lane * 16u;
        const char* src[C::PER];
        size_t step[C::PER];
#pragma unroll
        for (int i = 0; i < C::PER; ++i) {
            // fragment id of the stage: K step, then value, residual and weight tiles
            const int id = lw * C::PER + i, k = id / C::NX, x = id % C::NX;
            if (x < C::BM * C::XF) {
                const char* base = (const char*)(x < C::BM ? a.xhi : a.xlo);
                src[i] = base + ((size_t)k * a.MT + min(mt0 + x % C::BM, a.MT - 1)) * 1024;
                step[i] = (size_t)KST * a.MT * 1024;
            } else {
                src[i] = (const char*)a.w + ((size_t)min(nt0 + x - C::BM * C::XF, a.n_tiles - 1) * kb + k) * 1024;
                step[i] = KST * 1024;
            }
        }
        auto issue = [&](int slot) {
            unsigned char* dst = ring + (size_t)slot * C::STAGE + (size_t)lw * C::PER * 1024;
#pragma unroll
            for (int i = 0; i < C::PER; ++i) {
                __builtin_amdgcn_global_load_lds((const void*)(src[i] + loff), (lds)(dst + i * 1024), 16, 0, 0);
                src[i] += step[i];
            }
        };
#pragma unroll
        for (int s = 0; s < RING - 1; ++s)
            if (s < n_st) issue(s);
        int slot = RING - 1;
        for (int it = 0; it < n_st; ++it) {
            // the loads of the stages after `it` may stay in flight
            const int left = min(n_st - 1 - it, RING - 2);
#define WAIT(N) if (left == N) asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(RING - 2 >= N ? N * C::PER : 0) : "memory")
            WAIT(0);
            else WAIT(1);
            else WAIT(2);
            else WAIT(3);
            else WAIT(4);
#undef WAIT
            if (it + RING - 1 < n_st) issue(slot);
            slot = slot + 1 == RING ? 0 : slot + 1;
        }
        if (ARG) lds_sync();
        return;
    }

    // the rows' sum-of-squares partials, NSL slices per row, while the first
    // fragments are on their way
    if (a.n_sq > 0) {
        const int r = threadIdx.x % ROWS, sl = threadIdx.x / ROWS;
        if (sl < NSL) {
            const int m = min(mt0 * 16 + r, a.M - 1);
            float sm = 0.f;
#pragma unroll 8
            for (int p = sl; p < a.n_sq; p += NSL) sm += a.sq[(size_t)p * a.sq_stride + m];
            s_part[sl][r] = sm;
        }
    }
    const int wm = wid % WM, wn = wid / WM;
    f32x4 acc[TM][TN];
#pragma unroll
    for (int j = 0; j < TM; ++j)
#pragma unroll
        for (int i = 0; i < TN; ++i) acc[j][i] = f32x4{0.f, 0.f, 0.f, 0.f};
    int slot = 0;
    for (int it = 0; it < n_st; ++it) {
        lds_sync();
        const unsigned char* st = ring + (size_t)slot * C::STAGE + lane * 16;
#pragma unroll
        for (int k = 0; k < KST; ++k) {
            const unsigned char* sx = st + (size_t)(k * C::NX + wm * TM) * 1024;
            const unsigned char* sw = st + (size_t)(k * C::NX + C::BM * C::XF + wn * TN) * 1024;
            uint4 w[TN], xh[TM], xl[PAIR ? TM : 1];
#pragma unroll
            for (int i = 0; i < TN; ++i) w[i] = *(const uint4*)(sw + i * 1024);
#pragma unroll
            for (int j = 0; j < TM; ++j) {
                xh[j] = *(const uint4*)(sx + j * 1024);
                if (PAIR) xl[j] = *(const uint4*)(sx + (C::BM + j) * 1024);
            }
#pragma unroll
            for (int j = 0; j < TM; ++j)
#pragma unroll
                for (int i = 0; i < TN; ++i) {
                    if (PAIR) {
                        mma_frag<bf16>(acc[j][i], w[i], xh[j]);
                        mma_frag<bf16>(acc[j][i], w[i], xl[j]);
                    } else {
                        acc[j][i] = __builtin_amdgcn_mfma_f32_16x16x32_f16(
                            __builtin_bit_cast(f16x8, w[i]), __builtin_bit_cast(f16x8, xh[j]), acc[j][i], 0, 0, 0);
                    }
                }
        }
        slot = slot + 1 == RING ? 0 : slot + 1;
    }
    mfma_settle();
    const int mw = mt0 + wm * TM, nw = nt0 + wn * TN;          // the wave's first tiles
    if (!ARG && a.lrt > 0) {
        // LoRA expand of u [M][ldu], two rank tiles a product (lane group g
        // takes entries 4 g .. 4 g + 3 of either), u as bf16 value + residual.
        // Every source of the wave's tiles in turn: tiles (q/k/v) or tile rows
        // (gate/up: 0-7 gate, 8-15 up) of another take no part.
        const bool half = a.lora_mode == LORA_ROW_HALF;
        const int s_lo = half ? 0 : lora_src(a, nw), s_hi = half ? 1 : lora_src(a, min(nw + TN, a.n_tiles) - 1);
        for (int sc = s_lo; sc <= s_hi; ++sc)
            for (int t = 0; t < a.lrt; t += 2) {
                const bool two = t + 1 < a.lrt;
                bf16x8 bv[TN];
#pragma unroll
                for (int i = 0; i < TN; ++i) {
                    const int nt = min(nw + i, a.n_tiles - 1);
                    const uint2* lb = (const uint2*)a.lb + ((size_t)nt * a.lrt + t) * WAVE + lane;
                    uint2 b0 = lb[0], b1 = lb[two ? WAVE : 0];
                    const bool mine = half ? (lrow < 8) == (sc == 0) : lora_src(a, nt) == sc;
                    if (!mine) b0 = uint2{0u, 0u};
                    if (!mine || !two) b1 = uint2{0u, 0u};
                    bv[i] = __builtin_bit_cast(bf16x8, uint4{b0.x, b0.y, b1.x, b1.y});
                }
#pragma unroll
                for (int j = 0; j < TM; ++j) {
                    const int m = min((mw + j) * 16 + lrow, a.M - 1);
                    const float lsc = m % a.W >= a.adapter_from ? a.scale : 0.f;
                    const float* up = a.u + (size_t)m * a.ldu + (size_t)(sc * a.lrt + t) * 16 + lgrp * 4;
                    const float4 u0 = *(const float4*)up, u1 = *(const float4*)(up + (two ? 16 : 0));
                    const float uv[8] = {u0.x, u0.y, u0.z, u0.w, u1.x, u1.y, u1.z, u1.w};
                    bf16x8 h, l;
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        const float v = uv[e] * lsc;
                        h[e] = (bf16)v;
                        l[e] = (bf16)(v - (float)h[e]);
                    }
#pragma unroll
                    for (int i = 0; i < TN; ++i) {
                        acc[j][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bv[i], h, acc[j][i], 0, 0, 0);
                        acc[j][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bv[i], l, acc[j][i], 0, 0, 0);
                    }
                }
            }
        mfma_settle();
    }
#pragma unroll
    for (int j = 0; j < TM; ++j) {
        const int mt = mw + j, m = mt * 16 + lrow, r = (wm * TM + j) * 16 + lrow;
        float rm = 1.f;
        if (a.n_sq > 0) {
            float sm = 0.f;
#pragma unroll
            for (int sl = 0; sl < NSL; ++sl) sm += s_part[sl][r];
            rm = rsqrtf(sm / (float)a.norm_dim + a.eps);
        }
        if (ARG) {
            // logits, and the row's best over the wave's columns (the lowest
            // column wins ties) with its softmax partial
            const int excl = m % a.W >= a.excl_from ? a.exclude : -1;
            float best = -INFINITY, mx = -INFINITY, sm = 0.f;
            int bi = 0x7fffffff;
#pragma unroll
            for (int i = 0; i < TN; ++i) {
                const int nt = nw + i, col0 = nt * 16 + lgrp * 4;
                acc[j][i] *= rm;
                if (nt >= a.n_tiles) continue;
                const f32x4 v = acc[j][i];
                if (m < a.M && a.logits) *(float4*)(a.logits + (size_t)m * a.ldo + col0) = float4{v[0], v[1], v[2], v[3]};
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    if (col0 + e != excl && v[e] > best) { best = v[e]; bi = col0 + e; }
                    mx = fmaxf(mx, v[e]);
                }
            }
#pragma unroll
            for (int off = 16; off <= 32; off *= 2) {          // the row's four lane groups
                const float ob = __shfl_xor(best, off);
                const int oi = __shfl_xor(bi, off);
                if (ob > best || (ob == best && oi < bi)) { best = ob; bi = oi; }
            }
            if (a.arg_mx) {
                mx = fmaxf(mx, __shfl_xor(mx, 16));
                mx = fmaxf(mx, __shfl_xor(mx, 32));
                if (mx > -INFINITY) {
#pragma unroll
                    for (int i = 0; i < TN; ++i) {
                        if (nw + i >= a.n_tiles) continue;
#pragma unroll
                        for (int e = 0; e < 4; ++e) sm += expf(acc[j][i][e] - mx);
                    }
                }
                sm += __shfl_xor(sm, 16);
                sm += __shfl_xor(sm, 32);
            }
            if (lgrp == 0) {
                s_am[wn][0][ARG ? r : 0] = best;
                s_am[wn][1][ARG ? r : 0] = mx;
                s_am[wn][2][ARG ? r : 0] = sm;
                s_ai[wn][ARG ? r : 0] = bi;
            }
        } else {
            Resid res[TN];
#pragma unroll
            for (int i = 0; i < TN; ++i) res[i].load(a, m, nw + i, m < a.M && nw + i < a.n_tiles, lgrp);
#pragma unroll
            for (int i = 0; i < TN; ++i) {
                if (mt >= a.MT || nw + i >= a.n_tiles) continue;
                const f32x4 v = acc[j][i] * rm;
                put_tile<PAIR>(a, v, m, nw + i, m < a.M, lgrp, res[i]);
            }
        }
    }
    if (!ARG) return;
    lds_sync();
    // the block's partial of a row over its wave columns, in column order
    const int r = threadIdx.x, m = mt0 * 16 + r;
    if (r < ROWS && m < a.M) {
        float best = -INFINITY, mx = -INFINITY;
        int bi = 0x7fffffff;
#pragma unroll
        for (int w = 0; w < WN; ++w) {
            const float v = s_am[w][0][ARG ? r : 0];
            if (v > best) { best = v; bi = s_ai[w][ARG ? r : 0]; }
            mx = fmaxf(mx, s_am[w][1][ARG ? r : 0]);
        }
        a.arg_val[(size_t)bn * a.M + m] = best;
        a.arg_idx[(size_t)bn * a.M + m] = bi;
        if (a.arg_mx) {
            float sm = 0.f;
#pragma unroll
            for (int w = 0; w < WN; ++w) {
                const float pm = s_am[w][1][ARG ? r : 0];
                if (pm > -INFINITY) sm += s_am[w][2][ARG ? r : 0] * expf(pm - mx);
            }
            a.arg_mx[(size_t)bn * a.M + m] = mx;
            a.arg_sum[(size_t)bn * a.M + m] = sm;
        }
    }
}

template <bool PAIR, int WM, int WN, int TM, int TN, int NL, int KST, int RING, bool ARG>
hipError_t launch_tl(BigGemmArgs a, hipStream_t st) {
    typedef TL<PAIR, WM, WN, TM, TN, NL, KST, RING> C;
    a.gm = (a.MT + C::BM - 1) / C::BM;
    a.gn = (a.n_tiles + C::BN - 1) / C::BN;
    a.xmap = xcd_map(a);
    PBD_LAUNCH((k_gemm_tile<PAIR, WM, WN, TM, TN, NL, KST, RING, ARG>), dim3(xcd_grid(a)), dim3((C::NC + NL) * 64), C::LDS, st, a);
    return hipGetLastError();
}

#define TLI(P, WM, WN, TM, TN, NL, KST, RING, ARG) \
    {P, WM * TM, WN * TN, TM * TN, ARG, launch_tl<P, WM, WN, TM, TN, NL, KST, RING, ARG>}
// two K steps a stage where the stage is small (fewer barriers), one with a
// deeper ring where two would leave room for two stages only
const TileInst INST[] = {
    TLI(0, 2, 4, 2, 2, 4, 2, 4, 0), TLI(0, 2, 4, 4, 2, 4, 2, 4, 0), TLI(0, 2, 4, 5, 2, 4, 2, 3, 0),
    TLI(0, 2, 4, 6, 2, 4, 2, 3, 0), TLI(0, 2, 4, 4, 4, 4, 2, 3, 0),
    TLI(1, 2, 4, 2, 2, 4, 2, 3, 0), TLI(1, 2, 4, 4, 2, 4, 2, 3, 0), TLI(1, 2, 4, 4, 3, 4, 1, 5, 0),
    TLI(1, 2, 4, 2, 4, 4, 1, 6, 0), TLI(1, 2, 4, 3, 4, 4, 1, 5, 0),
    // LM heads
    TLI(0, 2, 4, 6, 3, 4, 2, 3, 1), TLI(0, 2, 4, 5, 4, 2, 1, 5, 1), TLI(1, 2, 4, 2, 4, 4, 1, 6, 1),
    TLI(1, 2, 4, 3, 4, 4, 1, 5, 1),
};
#undef TLI

}  // namespace

const TileInst* tile_insts(int* n) {
    *n = (int)(sizeof(INST) / sizeof(INST[0]));
    return INST;
}

}  // namespace pbd
