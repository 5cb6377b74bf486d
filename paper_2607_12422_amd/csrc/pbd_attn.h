// Device pieces shared by the attention kernels (bf16, head_dim 128 unless a
// template says otherwise): the LDS ring of key stages and its loader wave, one
// stage's scores, softmax and P.V on MFMA, and the cache-warming work-groups.
#pragma once

#include "pbd_device.h"
#include "pbd_kernels.h"

namespace pbd {

// The running maximum is raised (and the output rescaled) only when a score
// exceeds it by more than this (log2 units)
constexpr float RESCALE_SLACK = 8.f;
// ... in k_attn_rows.  A key at the maximum has the weight 1, which bf16 holds
// exactly, and the largest weights carry the rounding error of the sum.  k_attn has
// four maxima a split (and k_attn_chunk a block), one per wave; the one of
// k_attn_rows has to follow its keys closer to be as near to float64: with 8 the
// passes of up to three query tiles were 0.6 to 1.8 % further off than on k_attn,
// with 1 they are 0 to 1.3 % nearer (error of logits against float64, two layers,
// 2 to 16 sequences), in up to 0.4 % more time; with 0.5 0.1 to 1.7 %, in 0.3 to
// 0.6 % more.
constexpr float ROWS_SLACK = 1.f;

// 32 keys in LDS: two 16-key blocks of the cache, each 4 KiB of K then 4 KiB of V
constexpr int ATTN_STAGE = 16384;

// Work-groups past the splits warm the memory-side cache with what the next
// kernels read (the attention keeps few CUs busy): one word per 128-byte line
// of this work-group's share of the three ranges.
static __device__ __forceinline__ void attn_warm(const AttnArgs& a) {
    const int n_pf = (gridDim.x - a.s_launch) * gridDim.y * gridDim.z;
    const int ip = ((blockIdx.x - a.s_launch) * gridDim.y + blockIdx.y) * gridDim.z + blockIdx.z;
    const size_t n0 = a.pf_bytes[0] / 128, n1 = a.pf_bytes[1] / 128, n2 = a.pf_bytes[2] / 128;
    const size_t lines = n0 + n1 + n2;
    const size_t per = (lines + n_pf - 1) / n_pf;
    const size_t l0 = (size_t)ip * per, l1 = min(l0 + per, lines);
    constexpr int PFN = 16;
    unsigned v[PFN];
#pragma unroll
    for (int i = 0; i < PFN; ++i) {
        const size_t li = l0 + (size_t)i * blockDim.x + threadIdx.x;
        const char* p = li < n0 ? a.pf[0] + li * 128
                      : li < n0 + n1 ? a.pf[1] + (li - n0) * 128 : a.pf[2] + (li - n0 - n1) * 128;
        v[i] = li < l1 ? *(const unsigned*)p : 0u;
    }
    unsigned acc = 0;
#pragma unroll
    for (int i = 0; i < PFN; ++i) acc ^= v[i];
    asm volatile("" ::"v"(acc));
}

// The loader wave: stages 0 .. n_st - 1 of NB key blocks each, from block kb0
// on (no block past kb_last is read: it is repeated, its keys are masked), into
// the ring, RING - 1 stages ahead.  kc, vc: the head's cache plus 16 bytes per
// lane.  `before` runs once the first loads are on their way.  Takes part in
// one barrier per stage, which opens that stage.
template <int RING, int NB, typename BEFORE>
static __device__ __forceinline__ void attn_loader(const char* kc, const char* vc, int kb0, int kb_last, int n_st,
                                                   unsigned char* ring, BEFORE before) {
    typedef __attribute__((address_space(3))) void* lds;
    static_assert(RING >= 2 && RING <= 5 && 8 * NB * (RING - 2) < 64, "loads in flight fit the wait counter");
    auto issue = [&](int st, int slot) {
        unsigned char* dst = ring + (size_t)slot * NB * 8192;
#pragma unroll
        for (int c = 0; c < NB; ++c) {
            const size_t off = (size_t)min(kb0 + NB * st + c, kb_last) * 4096;
#pragma unroll
            for (int i = 0; i < 4; ++i)
                __builtin_amdgcn_global_load_lds((const void*)(kc + off + i * 1024), (lds)(dst + c * 8192 + i * 1024),
                                                 16, 0, 0);
#pragma unroll
            for (int i = 0; i < 4; ++i)
                __builtin_amdgcn_global_load_lds((const void*)(vc + off + i * 1024),
                                                 (lds)(dst + c * 8192 + 4096 + i * 1024), 16, 0, 0);
        }
    };
#pragma unroll
    for (int s = 0; s < RING - 1; ++s)
        if (s < n_st) issue(s, s);
    before();
    int slot = RING - 1;
    for (int it = 0; it < n_st; ++it) {
        // 8 NB loads a stage; those of the stages after `it` may stay in flight
        const int left = min(n_st - 1 - it, RING - 2);
        if (left >= 3) asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(RING >= 5 ? 24 * NB : 0) : "memory");
        else if (left == 2) asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(RING >= 4 ? 16 * NB : 0) : "memory");
        else if (left == 1) asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(RING >= 3 ? 8 * NB : 0) : "memory");
        else asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");
        // the stage read last turn (before this barrier) gives its slot
        if (it + RING - 1 < n_st) issue(it + RING - 1, slot);
        slot = slot + 1 == RING ? 0 : slot + 1;
    }
}

// One stage of 32 keys for TQ tiles of 16 query rows of a wave: S^T = K Q^T,
// online softmax per query column (exp2 domain) and O^T += V^T P^T with P^T
// straight from the score accumulators.  The products over both key blocks
// share one MFMA: its lane group g takes keys 4g .. 4g + 3 of either block, in
// the values as in the weights.  slack: how far a score may exceed the maximum
// before it is raised.  masked: some (key, row) pairs are not seen;
// ok(q, i): key i of the stage is seen by the lane's column of tile q.
template <int TQ, typename OK>
static __device__ __forceinline__ void attn_keys32(const unsigned char* st, int lane, const uint4 (&qf)[TQ][4],
                                                   f32x4 (&o)[TQ][8], float (&m)[TQ], float (&l)[TQ], bool first,
                                                   float slack, bool masked, OK ok) {
    const int lgrp = lane / 16;
    f32x4 sc[TQ][2];
#pragma unroll
    for (int q = 0; q < TQ; ++q) sc[q][0] = sc[q][1] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ds = 0; ds < 4; ++ds)
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const uint4 kf = *(const uint4*)(st + c * 8192 + ds * 1024 + lane * 16);
#pragma unroll
            for (int q = 0; q < TQ; ++q) mma_frag<bf16>(sc[q][c], kf, qf[q][ds]);
        }
    // explicit wait states before the scores are read: the compiler's own do
    // not cover the path that branches around the key mask
    mfma_settle();
    if (masked) {
#pragma unroll
        for (int q = 0; q < TQ; ++q)
#pragma unroll
            for (int c = 0; c < 2; ++c)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (!ok(q, c * 16 + lgrp * 4 + e)) sc[q][c][e] = -INFINITY;
    }
    bool over = first;
#pragma unroll
    for (int q = 0; q < TQ; ++q) {
        const float lim = m[q] + slack;
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int e = 0; e < 4; ++e) over = over | (sc[q][c][e] > lim);
    }
    if (__any(over)) {
#pragma unroll
        for (int q = 0; q < TQ; ++q) {
            float mloc = -1e30f;
#pragma unroll
            for (int c = 0; c < 2; ++c)
#pragma unroll
                for (int e = 0; e < 4; ++e) mloc = fmaxf(mloc, sc[q][c][e]);
            const float m_new = fmaxf(m[q], xrow_max(mloc));
            const float corr = __builtin_amdgcn_exp2f(m[q] - m_new);
            l[q] *= corr;
#pragma unroll
            for (int dt = 0; dt < 8; ++dt) o[q][dt] *= corr;
            m[q] = m_new;
        }
    }
    bf16x8 p[TQ];
#pragma unroll
    for (int q = 0; q < TQ; ++q)
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float w = __builtin_amdgcn_exp2f(sc[q][c][e] - m[q]);
                l[q] += w;
                p[q][c * 4 + e] = (bf16)w;
            }
#pragma unroll
    for (int dt = 0; dt < 8; ++dt) {
        const uint2 v0 = *(const uint2*)(st + 4096 + dt * 512 + lane * 8);
        const uint2 v1 = *(const uint2*)(st + 8192 + 4096 + dt * 512 + lane * 8);
        const bf16x8 v = __builtin_bit_cast(bf16x8, uint4{v0.x, v0.y, v1.x, v1.y});
#pragma unroll
        for (int q = 0; q < TQ; ++q) o[q][dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(v, p[q], o[q][dt], 0, 0, 0);
    }
    // and before anything may take the chain's source registers over
    mfma_settle();
}

}  // namespace pbd
