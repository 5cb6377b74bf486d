// Projection GEMM of bf16 models: K split over the waves of a work-group.  (At
// most two m-tiles with more rank tiles stay on the skinny GEMM; passes of many
// rows take the LDS blocks of pbd_tile.hip where gemm_pick says so.)
//
//   Y[m][n] = r_m * ( sum_k W[n][k] X[m][k]  +  s * sum_j B[n][j] u[m][j] ),
//   u[m][j] = sum_k A[j][k] X[m][k]                    (LoRA, adapter on)
//
// A work-group owns MB x NB 16 x 16 output tiles; wave w of its NW waves takes
// the K fragments w, w + NW, .. of all of them.  Operands and weights are
// packed fragment by fragment (1 KiB a wave load), so a wave needs nothing
// from its neighbours until the end: each fragment goes straight from the
// cache to the registers of the one wave that uses it (MB * NB MFMAs per
// MB + NB loads), PF steps ahead, with no LDS traffic and no barrier in the
// loop.  The waves' partial tiles are then summed in wave order through LDS,
// and the tiles' epilogues are shared out among the waves.  Small blocks and
// the split of K fill the chip where 64 x 64 blocks over the whole K leave it
// idle (48 of them for o and down at 136 rows, each a chain of 64 or 96 steps):
// at the Qwen3-0.6B shape, weights cold, q/k/v, o, gate/up and down take 8.4,
// 6.3, 9.3 and 7.8 us at 136 rows (64 x 64 blocks: 10.9, 13.6, 11.6, 19.3) and
// 7.7, 6.6, 9.8 and 8.4 us at 68 rows of value + residual operands (12.3, 17.2,
// 12.7, 24.3; the skinny GEMM 10.9, 18.8, 18.1, 18.8 in the pass).
#include "pbd_epi.h"
#include "pbd_launch.h"

#include <algorithm>

namespace pbd {
namespace {

// One tile of the LM head: logits, and per row (into am / ai, lanes of group
// 0) the best value and its column, and with confidence the maximum and the
// sum of exp(value - maximum) over the 16 columns.
__device__ __forceinline__ void arg_tile(const BigGemmArgs& a, const f32x4& v, int m, int nt, bool live, int lrow,
                                         int lgrp, float (*am)[16], int* ai) {
    const int col0 = nt * 16 + lgrp * 4;
    if (live && a.logits) *(float4*)(a.logits + (size_t)m * a.ldo + col0) = float4{v[0], v[1], v[2], v[3]};
    const int excl = m % a.W >= a.excl_from ? a.exclude : -1;
    float best = -INFINITY;
    int bi = 0x7fffffff;
#pragma unroll
    for (int e = 0; e < 4; ++e)
        if (col0 + e != excl && v[e] > best) { best = v[e]; bi = col0 + e; }   // ascending: first max wins
#pragma unroll
    for (int off = 16; off <= 32; off *= 2) {                    // the row's four lane groups
        const float ob = __shfl_xor(best, off);
        const int oi = __shfl_xor(bi, off);
        if (ob > best || (ob == best && oi < bi)) { best = ob; bi = oi; }
    }
    float mx = -INFINITY, sm = 0.f;
    if (a.arg_mx) {
        mx = fmaxf(fmaxf(v[0], v[1]), fmaxf(v[2], v[3]));
        mx = fmaxf(mx, __shfl_xor(mx, 16));
        mx = fmaxf(mx, __shfl_xor(mx, 32));
        sm = expf(v[0] - mx) + expf(v[1] - mx) + expf(v[2] - mx) + expf(v[3] - mx);
        sm += __shfl_xor(sm, 16);
        sm += __shfl_xor(sm, 32);
    }
    if (lgrp == 0) {
        am[0][lrow] = best;
        am[1][lrow] = mx;
        am[2][lrow] = sm;
        ai[lrow] = bi;
    }
}

// The block's partial of one row over its n tiles (am, ai: the row's column of
// each tile; ascending tiles, so that the lowest column wins ties).
__device__ __forceinline__ void arg_row(const BigGemmArgs& a, int m, int bn, int n, const float (*am)[3][16],
                                        const int (*ai)[16], int r) {
    float best = -INFINITY, mx = -INFINITY;
    int bi = 0x7fffffff;
    for (int i = 0; i < n; ++i) {
        const float v = am[i][0][r];
        if (v > best) { best = v; bi = ai[i][r]; }
        mx = fmaxf(mx, am[i][1][r]);
    }
    a.arg_val[(size_t)bn * a.M + m] = best;
    a.arg_idx[(size_t)bn * a.M + m] = bi;
    if (a.arg_mx) {
        float sm = 0.f;
        if (mx > -INFINITY)
            for (int i = 0; i < n; ++i)
                if (am[i][1][r] > -INFINITY) sm += am[i][2][r] * expf(am[i][1][r] - mx);
        a.arg_mx[(size_t)bn * a.M + m] = mx;
        a.arg_sum[(size_t)bn * a.M + m] = sm;
    }
}

constexpr int RED_KIB = 64;      // LDS of the cross-wave sum

// PAIR: bf16 value + residual operands against bf16 weights (two MFMAs per
// weight fragment); else fp16 operands and weights.  ST: LoRA A tiles whose
// shrink runs beside the projection (0: no adapter, or the shrink comes from
// a.u).
template <bool PAIR, int MB, int NB, int NW, int ST> struct GK {
    static constexpr int XF = PAIR ? 2 : 1;
    static constexpr int PER = 4 * (NB + MB * XF + ST);          // registers of one K step's fragments
    static constexpr int ACC = 4 * (MB * NB + MB * ST);
    // K steps in flight: two waves a SIMD leave 256 registers per lane
    static constexpr int PF = (208 - ACC) / PER >= 4 ? 4 : (208 - ACC) / PER >= 2 ? 2 : 1;
    static constexpr bool HALVES = NW * MB * NB > RED_KIB;       // the sum takes two rounds
    static_assert(NW * MB * NB <= 2 * RED_KIB, "cross-wave sum fits the LDS");
};

template <bool PAIR, int MB, int NB, int NW, int ST>
__global__ __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(2, 8))) void k_gemm_ks(BigGemmArgs a) {
    typedef GK<PAIR, MB, NB, NW, ST> C;
    constexpr int PF = C::PF, NT = MB * NB;
    const int lane = threadIdx.x % WAVE;
    const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE);
    const int lrow = lane % 16, lgrp = lane / 16;
    int bm, bn;
    if (!block_of(a, bm, bn)) return;
    const int mt0 = bm * MB, nt0 = bn * NB, kb = a.kb;
    __shared__ f32x4 s_red[C::HALVES ? NW / 2 : NW][NT][WAVE];
    __shared__ float s_part[8][MB * 16];
    // argmax: per tile and row the best value, the maximum and the sum of
    // exp(value - maximum) over the tile (blocks that can be an LM head's)
    constexpr bool ARG = NB == 4 && NW == 4 && ST == 0;
    __shared__ float s_am[ARG ? NT : 1][3][16];
    __shared__ int s_ai[ARG ? NT : 1][16];
    int ntc[NB], mtc[MB];
#pragma unroll
    for (int i = 0; i < NB; ++i) ntc[i] = min(nt0 + i, a.n_tiles - 1);
#pragma unroll
    for (int j = 0; j < MB; ++j) mtc[j] = min(mt0 + j, a.MT - 1);
    const u32x4* la = nullptr;
    if (ST > 0) {
        la = (const u32x4*)a.la + (size_t)lora_src(a, nt0) * ST * kb * WAVE;
    }
    u32x4 wv[PF][NB], xv[PF][MB * C::XF], av[PF][ST > 0 ? ST : 1];
    // K step i of this wave; steps past the end repeat the last fragment
    // (their products are not formed), so that every load is unconditional.
    // Uniform bases and one 32-bit lane offset: no vector address arithmetic.
    const unsigned loff = lane * 16u;
    const char* wb[NB];
#pragma unroll
    for (int n = 0; n < NB; ++n) wb[n] = (const char*)a.w + (size_t)ntc[n] * kb * 1024;
    auto load = [&](int i, int s) {
        const int f = min(wid + NW * i, kb - 1);
#pragma unroll
        for (int n = 0; n < NB; ++n) wv[s][n] = *(const u32x4*)(wb[n] + (size_t)f * 1024 + loff);
        const size_t xf = (size_t)f * a.MT * 1024;
#pragma unroll
        for (int j = 0; j < MB; ++j) {
            xv[s][j] = *(const u32x4*)((const char*)a.xhi + xf + (size_t)mtc[j] * 1024 + loff);
            if (PAIR) xv[s][MB + j] = *(const u32x4*)((const char*)a.xlo + xf + (size_t)mtc[j] * 1024 + loff);
        }
#pragma unroll
        for (int t = 0; t < ST; ++t) av[s][t] = *(const u32x4*)((const char*)la + ((size_t)t * kb + f) * 1024 + loff);
    };
    f32x4 acc[MB][NB], uacc[ST > 0 ? ST : 1][MB];
#pragma unroll
    for (int j = 0; j < MB; ++j) {
#pragma unroll
        for (int i = 0; i < NB; ++i) acc[j][i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int t = 0; t < ST; ++t) uacc[t][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    auto one = [&](f32x4& c, const u32x4& w, int s, int j) {
        if (PAIR) {
            mma_frag<bf16>(c, __builtin_bit_cast(uint4, w), __builtin_bit_cast(uint4, xv[s][j]));
            mma_frag<bf16>(c, __builtin_bit_cast(uint4, w), __builtin_bit_cast(uint4, xv[s][MB + j]));
        } else {
            c = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, w), __builtin_bit_cast(f16x8, xv[s][j]),
                                                       c, 0, 0, 0);
        }
    };
    auto compute = [&](int s) {
#pragma unroll
        for (int j = 0; j < MB; ++j) {
#pragma unroll
            for (int i = 0; i < NB; ++i) one(acc[j][i], wv[s][i], s, j);
#pragma unroll
            for (int t = 0; t < ST; ++t) one(uacc[t][j], av[s][t], s, j);
        }
    };
    const int ni = (kb - wid + NW - 1) / NW;       // K steps of this wave (kb < NW: none for the last waves)
#pragma unroll
    for (int s = 0; s < PF; ++s) load(s, s);
    // LoRA expand blocks of the tiles, and the rows' sum-of-squares partials
    // (up to eight slices per row), requested behind the first steps
    uint2 bv[ST > 0 ? NB : 1][ST > 0 ? ST : 1];
    if (ST > 0) {
        const int lrt = a.lrt;
#pragma unroll
        for (int i = 0; i < NB; ++i)
#pragma unroll
            for (int t = 0; t < ST; ++t)
                bv[i][t] = *(const uint2*)((const bf16*)a.lb + (((size_t)ntc[i] * lrt + (t < lrt ? t : t - lrt)) * WAVE + lane) * 4);
    }
    constexpr int NSL = NW * WAVE / (MB * 16) < 8 ? NW * WAVE / (MB * 16) : 8;
    if (a.n_sq > 0) {
        const int r = threadIdx.x % (MB * 16), sl = threadIdx.x / (MB * 16);
        if (sl < NSL) {
            const int m = min(mt0 * 16 + r, a.M - 1);
            float sm = 0.f;
#pragma unroll 8
            for (int p = sl; p < a.n_sq; p += NSL) sm += a.sq[(size_t)p * a.sq_stride + m];
            s_part[sl][r] = sm;
        }
    }
    int i0 = 0;
    for (; i0 + PF < ni; i0 += PF) {
#pragma unroll
        for (int s = 0; s < PF; ++s) {
            compute(s);                             // i0 + s < ni
            // keep each step's loads right behind its products (the scheduler
            // would gather all products first and then wait for every load)
            __builtin_amdgcn_sched_barrier(0);
            load(i0 + PF + s, s);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
#pragma unroll
    for (int s = 0; s < PF; ++s)
        if (i0 + s < ni) compute(s);
    mfma_settle();
    // this wave's LoRA expand on its own partial u (the expand is linear)
    if (ST > 0) {
        const int lrt = a.lrt;
#pragma unroll
        for (int j = 0; j < MB; ++j) {
            const int m = (mt0 + j) * 16 + lrow;
            const float lsc = m % a.W >= a.adapter_from ? a.scale : 0.f;
#pragma unroll
            for (int t = 0; t < ST; ++t) {
                const f32x4 u = uacc[t][j] * lsc;
#pragma unroll
                for (int i = 0; i < NB; ++i) {
                    uint2 b = bv[i][t];
                    // gate/up tiles: rows 0-7 take source 0 (gate), 8-15 source 1 (up)
                    if (a.lora_mode == LORA_ROW_HALF && ((lrow < 8) != (t < lrt))) b = uint2{0u, 0u};
                    mma_k4_split(acc[j][i], b, u);
                }
            }
        }
        mfma_settle();
    }
    // sum over the waves (wave order; with HALVES wave w first takes w + NW / 2's tiles)
    if (C::HALVES) {
        if (wid >= NW / 2)
#pragma unroll
            for (int j = 0; j < MB; ++j)
#pragma unroll
                for (int i = 0; i < NB; ++i) s_red[wid - NW / 2][j * NB + i][lane] = acc[j][i];
        lds_sync();
        if (wid < NW / 2)
#pragma unroll
            for (int j = 0; j < MB; ++j)
#pragma unroll
                for (int i = 0; i < NB; ++i) s_red[wid][j * NB + i][lane] += acc[j][i];
    } else {
#pragma unroll
        for (int j = 0; j < MB; ++j)
#pragma unroll
            for (int i = 0; i < NB; ++i) s_red[wid][j * NB + i][lane] = acc[j][i];
    }
    // epilogues: tile tt to wave tt % NW; lane: row lrow of the m-tile,
    // columns 4 lgrp .. 4 lgrp + 3 of the n-tile
    Resid res[(NT + NW - 1) / NW];
#pragma unroll
    for (int tt0 = 0; tt0 < NT; tt0 += NW) {
        const int tt = tt0 + wid, m = (mt0 + tt / NB) * 16 + lrow, nt = nt0 + tt % NB;
        res[tt0 / NW].load(a, m, nt, tt < NT && m < a.M && nt < a.n_tiles, lgrp);
    }
    lds_sync();
#pragma unroll
    for (int tt0 = 0; tt0 < NT; tt0 += NW) {
        const int tt = tt0 + wid;
        const int j = tt / NB, i = tt % NB;
        const int mt = mt0 + j, nt = nt0 + i, m = mt * 16 + lrow;
        const bool live = tt < NT && mt < a.MT && m < a.M && nt < a.n_tiles;
        if (tt >= NT || mt >= a.MT || nt >= a.n_tiles) continue;
        f32x4 v = s_red[0][tt][lane];
#pragma unroll
        for (int w = 1; w < (C::HALVES ? NW / 2 : NW); ++w) v += s_red[w][tt][lane];
        if (ST == 0 && a.lrt > 0) {
            // LoRA expand of a shrink computed beforehand: u [M][ldu]
            const int s0 = lora_src(a, nt);
            const int nsrc = a.lora_mode == LORA_ROW_HALF ? 2 : 1;
            const float lsc = (live && m % a.W >= a.adapter_from) ? a.scale : 0.f;
            const float* up = a.u + (size_t)min(m, a.M - 1) * a.ldu + (size_t)s0 * a.lrt * 16 + lgrp * 4;
            for (int sc = 0; sc < nsrc; ++sc) {
                const bool zero = nsrc == 2 && ((lrow < 8) != (sc == 0));
                float4 uv[MAX_RT];
                uint2 b[MAX_RT];
#pragma unroll
                for (int t = 0; t < MAX_RT; ++t) {
                    const int tc = min(t, a.lrt - 1);
                    uv[t] = *(const float4*)(up + (sc * a.lrt + tc) * 16);
                    b[t] = *(const uint2*)((const bf16*)a.lb + (((size_t)nt * a.lrt + tc) * WAVE + lane) * 4);
                }
#pragma unroll
                for (int t = 0; t < MAX_RT; ++t)
                    if (t < a.lrt)
                        mma_k4_split(v, zero ? uint2{0u, 0u} : b[t], f32x4{uv[t].x, uv[t].y, uv[t].z, uv[t].w} * lsc);
            }
            mfma_settle();
        }
        float rm = 1.f;
        if (a.n_sq > 0) {
            float sm = 0.f;
#pragma unroll
            for (int sl = 0; sl < NSL; ++sl) sm += s_part[sl][j * 16 + lrow];
            rm = rsqrtf(sm / (float)a.norm_dim + a.eps);
        }
        v *= rm;
        if (ARG && a.arg_val) arg_tile(a, v, m, nt, live, lrow, lgrp, s_am[tt], s_ai[tt]);
        else put_tile<PAIR>(a, v, m, nt, live, lgrp, res[tt0 / NW]);
    }
    if (!ARG || !a.arg_val) return;
    __syncthreads();
    const int m = mt0 * 16 + (int)threadIdx.x;
    if ((int)threadIdx.x < MB * 16 && m < a.M) {
        const int j = threadIdx.x / 16;
        arg_row(a, m, bn, min(NB, a.n_tiles - nt0), &s_am[j * NB], &s_ai[j * NB], threadIdx.x % 16);
    }
}

template <bool PAIR, int MB, int NB, int NW, int ST>
hipError_t launch_ks(BigGemmArgs a, hipStream_t st) {
    a.gm = (a.MT + MB - 1) / MB;
    a.gn = (a.n_tiles + NB - 1) / NB;
    a.xmap = xcd_map(a);
    PBD_LAUNCH((k_gemm_ks<PAIR, MB, NB, NW, ST>), dim3(xcd_grid(a)), dim3(NW * 64), 0, st, a);
    return hipGetLastError();
}

// One instance: blocks of mb x nb tiles, nw waves, st shrink tiles
struct Inst {
    int pair, mb, nb, nw, st;
    hipError_t (*launch)(BigGemmArgs, hipStream_t);
};
#define KS(P, MB, NB, NW, ST) {P, MB, NB, NW, ST, launch_ks<P, MB, NB, NW, ST>}
#define KS_PAIR(ST) KS(1, 1, 1, 8, ST), KS(1, 2, 1, 8, ST), KS(1, 2, 2, 8, ST), KS(1, 3, 2, 8, ST), KS(1, 2, 4, 8, ST)
#define KS_F16(ST) \
    KS(0, 1, 1, 8, ST), KS(0, 2, 1, 8, ST), KS(0, 3, 1, 8, ST), KS(0, 2, 2, 8, ST), KS(0, 3, 2, 8, ST), KS(0, 2, 4, 8, ST)
const Inst INST[] = {
    KS(0, 1, 1, 8, 0), KS(0, 1, 2, 8, 0), KS(0, 2, 1, 8, 0), KS(0, 3, 1, 8, 0), KS(0, 2, 2, 8, 0),
    KS(0, 3, 2, 8, 0), KS(0, 4, 2, 8, 0), KS(0, 5, 2, 8, 0), KS(0, 4, 4, 8, 0), KS(0, 2, 4, 4, 0), KS(0, 4, 4, 4, 0),
    KS(0, 5, 4, 4, 0),
    KS(1, 1, 1, 8, 0), KS(1, 1, 2, 8, 0), KS(1, 2, 1, 8, 0), KS(1, 2, 2, 8, 0), KS(1, 3, 2, 8, 0), KS(1, 4, 2, 8, 0),
    KS(1, 2, 4, 8, 0), KS(1, 4, 4, 8, 0), KS(1, 4, 4, 4, 0), KS(1, 5, 4, 4, 0),
    KS_F16(1), KS_F16(2), KS_F16(4), KS_PAIR(1), KS_PAIR(2), KS_PAIR(4),
};
#undef KS
#undef KS_PAIR
#undef KS_F16

// Times (us) behind the choice of an instance, fitted to all of them at 34 to
// 4096 rows of the Qwen3-0.6B projections on 256 CUs.  They rank instances; what
// all of a launch's candidates pay alike (the logits' stores of an LM head: 327
// us estimated for 1056 rows, 414 measured) is left out.
//
// K-split blocks: a CU takes in 70 KiB of fragments a microsecond in its loop
// (fitted; over whole kernels the counters show 17 .. 41, 27 .. 46 requests in
// flight per CU at 310 .. 550 cycles, the MFMAs at most 38 % busy and hardly an L2
// stall: they name no single limit), 62 over rounds of two work-groups of four waves; one of those alone has its start and end to
// itself.  Eight waves fill a CU, so a second round starts after the first
// one's epilogue.
float ks_cost(const Inst& c, int n_tiles, int kb, int MT) {
    const long blocks = (long)((MT + c.mb - 1) / c.mb) * ((n_tiles + c.nb - 1) / c.nb);
    const float rounds = (float)((blocks + 255) / 256);
    const float kib = (float)kb * (c.nb + c.mb * (c.pair ? 2 : 1) + c.st);
    if (c.nw == 8) return 4.f + rounds * kib / 70.f + (rounds - 1.f) * 1.5f;
    return blocks <= 256 ? 7.5f + kib / (c.pair ? 55.f : 80.f) : 4.f + rounds * kib / 62.f;
}

// LDS blocks: the same loads (66 KiB a microsecond, 58 with operands in pairs,
// whose twice as many products cover less of them), and an epilogue that grows
// with the tiles of a wave and waits for the residual where there is one; one
// work-group a CU.  At 1056 fp16 rows gate/up take 21.9 us in 8 x 16 tiles
// (K-split: 28.6), q/k/v 16.8 in 10 x 8 (23.0), the LM head 414 in 12 x 12 or
// 10 x 16 (64 x 64 and 128 x 128 blocks staged through registers: 768); at 1024
// rows in pairs gate/up 27.5 in 8 x 12 (37.9) and q/k/v 18.8 in 8 x 8 (25.6).
// With a quarter of the work-groups that the chip holds (o at 512 rows: 21.4
// against 10.4) the K split stays.
float tile_cost(const TileInst& c, int n_tiles, int kb, int MT, bool resid) {
    const long blocks = (long)((MT + c.bm - 1) / c.bm) * ((n_tiles + c.bn - 1) / c.bn);
    const float rounds = (float)((blocks + 255) / 256);
    const float kib = (float)kb * (c.bn + c.bm * (c.pair ? 2 : 1));
    const float epi = (c.pair ? 0.4f : 0.25f) * c.wtiles + (resid ? 4.f : 1.5f);
    return 2.f + rounds * (kib / (c.pair ? 58.f : 66.f) + epi);
}

struct Pick {
    hipError_t (*launch)(BigGemmArgs, hipStream_t);
    int bm, bn;
    float us;
    bool lds;          // pbd_tile.hip's
    int nw;            // waves of a K-split block
};

// The LM head's K-split blocks (four waves, four tiles) and the LDS blocks
// made for it leave one argmax partial per row and block.
Pick gemm_pick(int pair, int st, int n_tiles, int kb, int MT, bool argmax, bool resid) {
    Pick best{};
    auto take = [&](const Pick& p) {
        if (!best.launch || p.us < best.us) best = p;
    };
    for (const Inst& c : INST)
        if (c.pair == pair && c.st == st && (!argmax || (c.nw == 4 && c.nb == 4)))
            take(Pick{c.launch, c.mb, c.nb, ks_cost(c, n_tiles, kb, MT), false, c.nw});
    int n = 0;
    const TileInst* ti = tile_insts(&n);
    for (int i = 0; i < n && st == 0 && kb % 2 == 0; ++i)
        if (ti[i].pair == pair && ti[i].arg == (argmax ? 1 : 0))
            take(Pick{ti[i].launch, ti[i].bm, ti[i].bn, tile_cost(ti[i], n_tiles, kb, MT, resid), true, 0});
    return best;
}

}  // namespace

int gemm_shrink_tiles(int pair, int nsrc, bool half, int lrt, int n_tiles, int kb, int MT, bool resid) {
    // LoRA shrink inside the projection (its A tiles beside the weights in every
    // block) or as a launch of its own, whose few blocks walk the whole K, and
    // 0.5 us for u's way through memory: whichever is less.  (4.5 us for any
    // launch took four layers of hidden 2560, one sequence, rank 16, from 530 us
    // a draft to 593: down's K of 9728 makes it 16.8 us.  Over 1 .. 32 sequences
    // of 8, 17 and 33 rows, ranks 8 .. 64, four layer shapes, no draft is more
    // than 2.4 % off the best of 0, 0.5, 1 and 1.5 us; with each of the others
    // one is 7 to 8 %.)
    const int st = half ? 2 * lrt : lrt;
    if (lrt <= 0 || !(st == 1 || st == 2 || st == 4)) return 0;
    const float in = gemm_pick(pair, st, n_tiles, kb, MT, false, resid).us;
    const float ext = gemm_pick(pair, 0, n_tiles, kb, MT, false, resid).us +
                      gemm_pick(pair, 0, nsrc * lrt, kb, MT, false, false).us + 0.5f;
    return in <= ext ? st : 0;
}

int gemm_rows_shrink_tiles(const BigGemmArgs& a) {
    const int nsrc = a.lora_mode == LORA_BY_TILE ? 3 : a.lora_mode == LORA_ROW_HALF ? 2 : 1;
    return gemm_shrink_tiles(a.op_f16 ? 0 : 1, nsrc, a.lora_mode == LORA_ROW_HALF, a.lrt, a.n_tiles, a.kb, a.MT, a.rx != nullptr);
}

int gemm_choice(int pair, int st, int n_tiles, int kb, int MT, bool argmax, bool resid, int* block) {
    const Pick c = gemm_pick(pair, st, n_tiles, kb, MT, argmax, resid);
    block[0] = c.lds ? 1 : 0; block[1] = c.bm; block[2] = c.bn; block[3] = c.nw;
    return c.launch ? 1 : 0;
}

int gemm_rows_parts(const BigGemmArgs& a) {
    const Pick c = gemm_pick(a.op_f16 ? 0 : 1, 0, a.n_tiles, a.kb, a.MT, true, false);
    return (a.n_tiles + c.bn - 1) / c.bn;
}

hipError_t launch_gemm_rows(const BigGemmArgs& a, hipStream_t st) {
    if (!a.arg_val && !a.sw_hi && !a.rx && !a.out) return hipErrorInvalidValue;   // no destination
    if (a.M < 1 || a.MT != (a.M + 15) / 16 || a.n_tiles < 1 || a.kb < 1) return hipErrorInvalidValue;
    if (a.op_f16 ? a.xlo != nullptr : a.xlo == nullptr) return hipErrorInvalidValue;
    int sh = 0;
    if (a.lrt > 0) {
        if (a.lrt > MAX_RT || !a.lb || a.W < 1) return hipErrorInvalidValue;
        if (a.la) sh = (a.lora_mode == LORA_ROW_HALF ? 2 : 1) * a.lrt;
        else if (!a.u) return hipErrorInvalidValue;
        // a block's tiles share their LoRA source (blocks of 1, 2 or 4 tiles)
        if (sh && a.lora_mode == LORA_BY_TILE && (a.tile_split0 % 4 || a.tile_split1 % 4)) return hipErrorInvalidValue;
    }
    const Pick c = gemm_pick(a.op_f16 ? 0 : 1, sh, a.n_tiles, a.kb, a.MT, a.arg_val != nullptr, a.rx != nullptr);
    return c.launch ? c.launch(a, st) : hipErrorInvalidValue;
}

}  // namespace pbd
