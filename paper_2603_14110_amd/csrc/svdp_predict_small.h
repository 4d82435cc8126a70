// Both predictor stages of one token in one launch, for layers whose P is a few tiles (k_xP + k_scores otherwise).
//
// Bound of the two launches there: the launches.  Every block of the scores forms t = x P by itself from at most
// PS_TILES tiles of P (16 or 32 KB each, from L2 after the first block) while its rows of Q are on their way.  All sums are
// formed in the order of k_xP and k_scores, so that the scores have the same bits (svdp_ffn_step_glued keeps those two).
// Measured, one step, two launches -> one (us, issued one by one / in a graph with 24 layers in turn): d = 256, r = 32, fp32
// (one tile) 18.2 -> 15.1 / 13.6 -> 10.5 (484 of 1024 rows listed; about 100 listed: 19.1 -> 15.5 one by one); d = 1024, r = 32,
// bf16 (four tiles) 17.6 -> 14.7 / 15.3 -> 14.2; with eight tiles (d = 2048, r = 32) a graph is slower, 15.6 -> 18.2, hence
// the limit.  A wide layer does not change that: d = 1024, D = 18944, r = 32, predictor alone 12.9 -> 9.9 / 6.6 -> 4.7.
#pragma once

#include "svdp_kernels.h"

namespace svdp {

constexpr int PS_THREADS = 512;
constexpr int PS_GROUPS = PS_THREADS / XP_THREADS;       // tiles of P worked on together
constexpr int PS_TILES = 4;

template <typename W>
constexpr int ps_tile_floats()                           // scratch of one tile's reduction
{
    return (XP_THREADS / (XP_COLS / Elem<W>::VEC)) * (XP_COLS + 1) + XP_THREADS;
}
template <typename W>
size_t ps_lds(int d, int r)
{
    const int nt = (d + XP_ROWS - 1) / XP_ROWS;
    return ((size_t)PS_GROUPS * ps_tile_floats<W>() + (size_t)(nt + 1) * r) * 4;
}

// One block per slab of 64 neurons.  r / VEC <= 2^LPR_LOG2.
template <typename W, int LPR_LOG2>
__global__ __launch_bounds__(PS_THREADS) void k_predict_small(const W *__restrict__ P, const W *__restrict__ Q,
                                                              const float *__restrict__ bias, const W *__restrict__ x, int d,
                                                              int r, float *__restrict__ s_out, uint64_t *__restrict__ mask_out)
{
    constexpr int VEC = Elem<W>::VEC, CG = XP_COLS / VEC, NSUB = XP_THREADS / CG, RPT = XP_ROWS / NSUB;
    constexpr int PARTS = XP_THREADS / XP_COLS, PER = NSUB / PARTS;
    constexpr int LPR = 1 << LPR_LOG2, NGRP = PS_THREADS / LPR, RPG = (SC_SLAB + NGRP - 1) / NGRP;
    extern __shared__ float smem[];
    __shared__ float sc[SC_SLAB];
    const int tid = threadIdx.x, i0 = blockIdx.x * SC_SLAB;
    const int nt = (d + XP_ROWS - 1) / XP_ROWS, ncs = (r + XP_COLS - 1) / XP_COLS;
    float *tp = smem + PS_GROUPS * ps_tile_floats<W>(), *ts = tp + nt * r;       // partials of t [nt][r], t [r]

    // this lane group's rows of Q and their bias
    const int lig = tid & (LPR - 1), row = tid >> LPR_LOG2;
    const bool cols = lig * VEC < r;
    uint4 qraw[RPG];
#pragma unroll
    for (int k = 0; k < RPG; ++k) {
        qraw[k] = make_uint4(0u, 0u, 0u, 0u);
        if (cols && row + k * NGRP < SC_SLAB) qraw[k] = load_raw(Q + (size_t)(i0 + row + k * NGRP) * r + lig * VEC);
    }
    const float my_bias = tid < SC_SLAB ? bias[i0 + tid] : 0.f;

    // tiles of P as k_xP: 256 threads each
    const int gt = tid % XP_THREADS, cgi = gt % CG, sub = gt / CG;
    float *red = smem + tid / XP_THREADS * ps_tile_floats<W>(), *red2 = red + NSUB * (XP_COLS + 1);
    for (int u0 = 0; u0 < nt * ncs; u0 += PS_GROUPS) {
        const int u = u0 + tid / XP_THREADS, j0 = u / ncs * XP_ROWS, c0 = u % ncs * XP_COLS, col = c0 + cgi * VEC;
        const bool on = u < nt * ncs, colok = on && col < r;
        uint4 raw[RPT];
        float xv[RPT], acc[VEC];
#pragma unroll
        for (int e = 0; e < VEC; ++e) acc[e] = 0.f;
#pragma unroll
        for (int k = 0; k < RPT; ++k) {
            const int j = j0 + sub + k * NSUB;
            raw[k] = make_uint4(0u, 0u, 0u, 0u);
            xv[k] = 0.f;
            if (colok && j < d) {
                raw[k] = load_raw(P + (size_t)j * r + col);
                xv[k] = to_f32(x[j]);
            }
        }
#pragma unroll
        for (int k = 0; k < RPT; ++k) {
            float w[VEC];
            widen(raw[k], w, (const W *)nullptr);
            if (colok && j0 + sub + k * NSUB < d) {
#pragma unroll
                for (int e = 0; e < VEC; ++e) acc[e] = fmaf(xv[k], w[e], acc[e]);
            }
        }
#pragma unroll
        for (int e = 0; e < VEC; ++e) red[sub * (XP_COLS + 1) + cgi * VEC + e] = acc[e];
        __syncthreads();
        {
            const int o = gt % XP_COLS, part = gt / XP_COLS;
            float s = 0.f;
#pragma unroll
            for (int q = 0; q < PER; ++q) s += red[(part * PER + q) * (XP_COLS + 1) + o];
            red2[part * XP_COLS + o] = s;
        }
        __syncthreads();
        if (on && gt < XP_COLS && c0 + gt < r) {
            float t = 0.f;
#pragma unroll
            for (int q = 0; q < PARTS; ++q) t += red2[q * XP_COLS + gt];
            tp[u / ncs * r + c0 + gt] = t;
        }
    }
    __syncthreads();
    for (int c = tid; c < r; c += PS_THREADS) {
        float t = tp[c];
        for (int g = 1; g < nt; ++g) t += tp[g * r + c];
        ts[c] = t;
    }
    __syncthreads();

    // scores as k_scores
    float tv[VEC];
#pragma unroll
    for (int e = 0; e < VEC; ++e) tv[e] = cols ? ts[lig * VEC + e] : 0.f;
#pragma unroll
    for (int k = 0; k < RPG; ++k) {
        float w[VEC], acc = 0.f;
        widen(qraw[k], w, (const W *)nullptr);
        if (cols) {
#pragma unroll
            for (int e = 0; e < VEC; ++e) acc = fmaf(tv[e], w[e], acc);
        }
        const float s = group_sum<LPR_LOG2>(acc);
        if (lig == 0 && row + k * NGRP < SC_SLAB) sc[row + k * NGRP] = s;
    }
    __syncthreads();
    if (tid < SC_SLAB) {
        const float s = sc[tid] + my_bias;
        if (s_out != nullptr) s_out[i0 + tid] = s;
        const uint64_t m = __ballot(s > 0.f);
        if (mask_out != nullptr && tid == 0) mask_out[blockIdx.x] = m;
    }
}

}   // namespace svdp
