// Pieces shared by the projection GEMMs of many rows (pbd_gemm.hip,
// pbd_tile.hip): the work-group to block mapping and the tiles' epilogues.
#pragma once

#include "pbd_device.h"
#include "pbd_kernels.h"

namespace pbd {

typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

enum { KS_XN = 0, KS_XW = 1, KS_XM = 2 };

// Work-group id -> (m-block, n-block); false: none.  Work-groups of one XCD
// (id % 8; its own L2) take every eighth n-block.  Their share of the weights
// stays in that L2 while the m-blocks go by (XN); weights too large for that
// go by once, every m-block of an n-block following on (XW).  With few
// n-blocks the XCDs share out the m-blocks (XM).
static __device__ __forceinline__ bool block_of(const BigGemmArgs& a, int& bm, int& bn) {
    const int xcd = blockIdx.x % 8, id = blockIdx.x / 8, gn8 = (a.gn + 7) / 8;
    bm = a.xmap == KS_XM ? (id / a.gn) * 8 + xcd : a.xmap == KS_XN ? id / gn8 : id % a.gm;
    bn = a.xmap == KS_XM ? id % a.gn : (a.xmap == KS_XN ? id % gn8 : id / a.gm) * 8 + xcd;
    return bm < a.gm && bn < a.gn;
}

static __device__ __forceinline__ int lora_src(const BigGemmArgs& a, int nt) {
    return a.lora_mode == LORA_BY_TILE ? (nt < a.tile_split0 ? 0 : nt < a.tile_split1 ? 1 : 2) : 0;
}

// What a tile's residual epilogue reads, requested ahead of it.
struct Resid {
    float4 x;
    uint2 g;
    __device__ __forceinline__ void load(const BigGemmArgs& a, int m, int nt, bool live, int lgrp) {
        x = float4{0.f, 0.f, 0.f, 0.f};
        g = uint2{0u, 0u};
        if (a.rx && live) {
            x = *(const float4*)(a.rx + (size_t)m * a.ldx + nt * 16 + lgrp * 4);
            g = *(const uint2*)((const bf16*)a.rgain + nt * 16 + lgrp * 4);
        }
    }
};

// One tile's store (v scaled by r_m; lane: row lrow = m % 16, columns 4 lgrp
// .. 4 lgrp + 3): q/k/v, the residual x += y with the next operand and the
// row's sum of squares, or SwiGLU.  Every lane of the wave takes part.
template <bool PAIR>
static __device__ __forceinline__ void put_tile(const BigGemmArgs& a, const f32x4& v, int m, int nt, bool live, int lgrp,
                                         const Resid& r) {
    const int col0 = nt * 16 + lgrp * 4;
    if (a.rx) {
        const float4 xo = r.x;
        float xv4[4] = {xo.x + v[0], xo.y + v[1], xo.z + v[2], xo.w + v[3]};
        if (!live) xv4[0] = xv4[1] = xv4[2] = xv4[3] = 0.f;
        if (live) *(float4*)(a.rx + (size_t)m * a.ldx + col0) = float4{xv4[0], xv4[1], xv4[2], xv4[3]};
        float ss = xv4[0] * xv4[0] + xv4[1] * xv4[1] + xv4[2] * xv4[2] + xv4[3] * xv4[3];
        ss += __shfl_xor(ss, 16);
        ss += __shfl_xor(ss, 32);
        const bf16x4 g = __builtin_bit_cast(bf16x4, r.g);
        float ov[8];                     // runs of eight values, four from the neighbouring lane group
#pragma unroll
        for (int e = 0; e < 4; ++e) ov[e] = xv4[e] * (float)g[e];
#pragma unroll
        for (int e = 0; e < 4; ++e) ov[4 + e] = __shfl_xor(ov[e], 16);
        if (live && (lgrp % 2) == 0)
            put_operand_run<bf16>((bf16*)a.rn_hi, (bf16*)a.rn_lo, xfrag_elem<bf16>(m, col0, a.rn_MT), ov, !PAIR);
        if (live && lgrp == 0) a.rsq[(size_t)nt * a.rsq_stride + m] = ss;
    } else if (a.sw_hi) {
        float h[8];                      // the lane's up values sit 32 lanes away (column + 8)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float gt = v[e], up = __shfl_xor(v[e], 32);
            h[e] = gt / (1.f + __expf(-gt)) * up;
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) h[4 + e] = __shfl_xor(h[e], 16);
        if (live && lgrp == 0)
            put_operand_run<bf16>((bf16*)a.sw_hi, (bf16*)a.sw_lo, xfrag_elem<bf16>(m, nt * 8, a.sw_MT), h, !PAIR);
    } else if (live) {
        *(float4*)(a.out + (size_t)m * a.ldo + col0) = float4{v[0], v[1], v[2], v[3]};
    }
}

inline int xcd_map(const BigGemmArgs& a) {
    // an eighth of the blocks to each XCD, by columns or by rows
    auto even = [](int n) { return n >= 8 && (n % 8 == 0 || n >= 64); };
    const size_t w = (size_t)a.n_tiles * a.kb * 1024, x = (size_t)a.MT * a.kb * (a.xlo ? 2048 : 1024);
    // by rows every XCD reads all the weights, by columns the whole operand: o
    // at 4096 rows in pairs (33 MB against 4), 8 x 8 tiles: 34 us by rows, 54
    // by columns; gate/up there (17 MB against 13), 8 x 12: 106 and 99
    if (!even(a.gn) || (even(a.gm) && x >= 2 * w)) return KS_XM;
    return w / 8 <= ((size_t)2 << 20) ? KS_XN : KS_XW;
}

// Grid of gm x gn blocks under that mapping
inline unsigned xcd_grid(const BigGemmArgs& a) {
    return a.xmap == KS_XM ? 8u * ((a.gm + 7) / 8) * a.gn : 8u * ((a.gn + 7) / 8) * a.gm;
}

// An instance of the LDS-tiled GEMM (pbd_tile.hip): blocks of bm x bn tiles,
// wtiles of them per wave; kb must be even
struct TileInst {
    int pair, bm, bn, wtiles, arg;
    hipError_t (*launch)(BigGemmArgs, hipStream_t);
};
const TileInst* tile_insts(int* n);

}  // namespace pbd
