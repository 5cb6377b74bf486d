// Attention of prefill chunks (bf16, head_dim 128).
//
// The chunk's keys and values are in the cache already (k_kvwrite).  A
// work-group takes 64 query rows of one KV head (a row: query head gi of the
// head's G, chunk row j) over every key they see and writes the O-projection
// operand directly: no split partials and no merge kernel.  Its eight computing
// waves are two pairs of query tiles by four quarters of each 128-key stage;
// a ninth wave streams the stages from the cache into a double buffer in LDS.
// Two tiles per wave halve the LDS reads per product (at one tile they take
// twice the MFMAs' time), and the split of the keys gives a SIMD two waves
// although a 1024-row chunk has only 256 such work-groups.  Blocks past the
// causal limit of the work-group's last row are not read, and a wave skips the
// stages past its own; rows past the prompt cost nothing.  41 us a layer, on
// average, for the four 1024-row chunks of a 4096-token prompt (k_attn's
// one-tile work-groups and the merge: 106 + 11) and 12 us for one 512-row chunk
// (23 + 5), where half the CUs have a work-group.
#include "pbd_attn.h"
#include "pbd_launch.h"

namespace pbd {
namespace {

constexpr int QW = 2, TQ = 2, KS = 4;             // pairs of tiles, tiles per wave, key quarters
constexpr int ROWS = QW * TQ * 16;                // query rows of a work-group
constexpr int NW = QW * KS;                       // computing waves
constexpr int KEYS = KS * 32;                     // keys of a stage
constexpr int LDQ = 128 + 8;
constexpr size_t RING_BYTES = 2 * (size_t)KS * ATTN_STAGE;
// the waves' partial outputs lie over the ring after the key loop
static_assert((size_t)NW * TQ * 8 * 1024 <= RING_BYTES, "partials fit the ring");
// the query rows over its second stage, filled once they are in registers
static_assert(ROWS * LDQ * 2 <= KS * ATTN_STAGE, "query rows fit a stage");

__global__ __launch_bounds__((NW + 1) * 64) __attribute__((amdgpu_waves_per_eu(3, 8))) void k_attn_chunk(AttnArgs a) {
    typedef bf16 T;
    constexpr int HD = 128, HALF = HD / 2, NDS = 4, NDT = 8;
    typedef RowPrep<T, HD> RP;
    extern __shared__ __align__(16) unsigned char smem[];      // [2][KS][ATTN_STAGE]
    __shared__ float s_ml[KS][ROWS][2];
    T* q_l = (T*)(smem + (size_t)KS * ATTN_STAGE);             // [ROWS][LDQ]

    // one KV head per XCD (id % 8) where there are eight: its keys stay in that L2
    const int g = blockIdx.x, b = blockIdx.z;
    const int q0 = (gridDim.y - 1 - blockIdx.y) * ROWS;        // longest causal rows first
    // uniform (a row's address must not wait for them in a branch of its own)
    const int t = __builtin_amdgcn_readfirstlane(a.pos0[b]), nrows = __builtin_amdgcn_readfirstlane(a.nrows[b]);
    const int W = a.W, G = a.G, QR = G * W;
    const int lane = threadIdx.x % WAVE, wid = __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE);
    const int lrow = lane % 16, lgrp = lane / 16;
    // first and last chunk row of query rows [qa, qa + n)
    auto row_lo = [&](int qa, int n) { return qa / W == min(qa + n - 1, QR - 1) / W ? qa % W : 0; };
    auto row_hi = [&](int qa, int n) {
        const int qe = min(qa + n - 1, QR - 1);
        return qa / W == qe / W ? qe % W : W - 1;
    };
    if (row_lo(q0, ROWS) >= nrows) {
        // no live row: zeros
        const int dim = threadIdx.x % 16 * 8;
        const float z[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        for (int i = threadIdx.x / 16; i < ROWS; i += (NW + 1) * 4) {
            const int q = q0 + i;
            if (q < QR)
                put_operand_run<T>((T*)a.op_hi, (T*)a.op_lo, xfrag_elem<T>(b * W + q % W, (g * G + q / W) * HD + dim, a.MT), z);
        }
        return;
    }
    const int k_end = t + min(nrows, row_hi(q0, ROWS) + 1);
    const int n_st = ceil_div(k_end, KEYS);
    const size_t head = (((size_t)a.layer * a.max_batch + b) * a.n_kv + g) * a.nblk * 16 * HD;

    if (wid == NW) {
        const char* kc = (const char*)((const T*)a.kcache + head) + lane * 16;
        const char* vc = (const char*)((const T*)a.vcache + head) + lane * 16;
        attn_loader<2, 2 * KS>(kc, vc, 0, ceil_div(k_end, 16) - 1, n_st, smem, [] { lds_sync(); });
        lds_sync();
        lds_sync();
        return;
    }
    // query rows: normed, rotated and scaled by log2 e / sqrt(head_dim)
    {
        Gains<T, HD> gq;
        if (a.qk_norm) gq.load(a.q_norm, lrow);
        RP rp[ROWS / (NW * 4)];
#pragma unroll
        for (int i = 0; i < ROWS / (NW * 4); ++i) {
            // dead rows read a valid row, at a position of the table
            const unsigned q = min(q0 + i * NW * 4 + wid * 4 + lgrp, QR - 1), gi = q / (unsigned)W;
            const int j = min((int)(q - gi * W), nrows - 1);
            rp[i].load(a.qkv + ((size_t)b * W + j) * a.nqkv + (size_t)(g * G + gi) * HD,
                       a.rope + (size_t)(t + j) * HALF, lrow);
        }
        float gq_lo[RP::NP], gq_hi[RP::NP];
        gq.get(a.qk_norm, gq_lo, gq_hi);
#pragma unroll
        for (int p = 0; p < RP::NP; ++p) {
            gq_lo[p] *= a.scale_log2;
            gq_hi[p] *= a.scale_log2;
        }
#pragma unroll
        for (int i = 0; i < ROWS / (NW * 4); ++i) {
            const int ql = i * NW * 4 + wid * 4 + lgrp;
            T lo[RP::NP], hi[RP::NP];
            rp[i].finish(q_l + ql * LDQ, q0 + ql < QR, gq_lo, gq_hi, a.qk_norm, a.eps, lrow, lo, hi);
        }
    }
    lds_sync();
    const int qw = wid % QW, ks = wid / QW;
    uint4 qf[TQ][NDS];
    int jq[TQ];
#pragma unroll
    for (int q = 0; q < TQ; ++q) {
        const int ql = (qw * TQ + q) * 16 + lrow;
        jq[q] = (q0 + ql) % W;
#pragma unroll
        for (int ds = 0; ds < NDS; ++ds) qf[q][ds] = *(const uint4*)(q_l + ql * LDQ + ds * 32 + lgrp * 8);
    }
    // keys every row of this wave sees, and the last one any of them sees
    const int qa = min(q0 + qw * TQ * 16, QR - 1);
    const int k_full = t + min(row_lo(qa, TQ * 16) + 1, nrows), k_last = t + row_hi(qa, TQ * 16);

    f32x4 o[TQ][NDT];
    float m[TQ], l[TQ];
#pragma unroll
    for (int q = 0; q < TQ; ++q) {
        m[q] = -1e30f;
        l[q] = 0.f;
#pragma unroll
        for (int dt = 0; dt < NDT; ++dt) o[q][dt] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    for (int it = 0; it < n_st; ++it) {
        lds_sync();
        const int k0 = it * KEYS + ks * 32;
        if (k0 > k_last || k0 >= k_end) continue;
        attn_keys32<TQ>(smem + (size_t)((it & 1) * KS + ks) * ATTN_STAGE, lane, qf, o, m, l, false, RESCALE_SLACK,
                        k0 + 32 > k_full, [&](int q, int i) { return (k0 + i < k_end) & (k0 + i - t <= jq[q]); });
    }

    // merge of the key quarters: every wave leaves its sums, then takes two of
    // the eight 16-dim tiles of its query tiles
#pragma unroll
    for (int q = 0; q < TQ; ++q) {
        l[q] = xrow_sum(l[q]);
        if (lgrp == 0) {
            s_ml[ks][(qw * TQ + q) * 16 + lrow][0] = m[q];
            s_ml[ks][(qw * TQ + q) * 16 + lrow][1] = l[q];
        }
    }
    lds_sync();                                    // every wave past its last stage
    f32x4* part = (f32x4*)smem;                    // [KS][QW][TQ][NDT][WAVE]
#pragma unroll
    for (int q = 0; q < TQ; ++q)
#pragma unroll
        for (int dt = 0; dt < NDT; ++dt) part[(((size_t)ks * QW + qw) * TQ + q) * NDT * WAVE + dt * WAVE + lane] = o[q][dt];
    lds_sync();
#pragma unroll
    for (int q = 0; q < TQ; ++q) {
        const int ql = (qw * TQ + q) * 16 + lrow, qi = q0 + ql;
        float f[KS], mx = -1e30f, L = 0.f;
#pragma unroll
        for (int k = 0; k < KS; ++k) mx = fmaxf(mx, s_ml[k][ql][0]);
#pragma unroll
        for (int k = 0; k < KS; ++k) {
            f[k] = exp2f(s_ml[k][ql][0] - mx);
            L += f[k] * s_ml[k][ql][1];
        }
        const float inv = L > 0.f ? 1.f / L : 0.f;
#pragma unroll
        for (int d = 0; d < NDT / KS; ++d) {
            const int dt = ks * (NDT / KS) + d;
            f32x4 v = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int k = 0; k < KS; ++k) v += part[(((size_t)k * QW + qw) * TQ + q) * NDT * WAVE + dt * WAVE + lane] * f[k];
            v *= inv;
            float ov[8];                           // runs of eight dims, four from the neighbouring lane group
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                ov[e] = v[e];
                ov[4 + e] = __shfl_xor(v[e], 16);
            }
            if (qi < QR && lgrp % 2 == 0)
                put_operand_run<T>((T*)a.op_hi, (T*)a.op_lo,
                                   xfrag_elem<T>(b * W + qi % W, (g * G + qi / W) * HD + dt * 16 + lgrp * 4, a.MT), ov);
        }
    }
}

}  // namespace

bool attn_chunk_fits(int dtype, int head_dim) { return dtype == PBD_DTYPE_BF16 && head_dim == 128; }

hipError_t launch_attn_chunk(const AttnArgs& a, int batch, hipStream_t st) {
    if (!a.chunk || !a.op_hi || a.W < 1 || a.MT * 16 < batch * a.W) return hipErrorInvalidValue;
    const dim3 grid(a.n_kv, (a.G * a.W + ROWS - 1) / ROWS, batch);
    PBD_LAUNCH(k_attn_chunk, grid, dim3((NW + 1) * 64), RING_BYTES, st, a);
    return hipGetLastError();
}

}  // namespace pbd
