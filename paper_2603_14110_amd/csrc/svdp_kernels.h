// gfx950 kernels of the sparse decode step.  Template parameters:
//   W  : storage element (float or bf16); arithmetic is always fp32
//   NB : compile-time batch capacity (1, 2, 4, 8); the runtime batch B <= NB
// Every floating-point sum below is formed in an order that depends only on
// the launch shape and the index list, never on timing (no fp atomics).
#pragma once

#include "svdp_device.h"

#include <type_traits>

namespace svdp {

constexpr size_t LDS_MAX = 160 * 1024;    // bytes of LDS of one gfx950 compute unit
constexpr int XP_THREADS = 256;      // k_xP block
constexpr int XP_ROWS = 256;         // rows of P per k_xP block
constexpr int XP_COLS = 32;          // columns of P per k_xP block
constexpr int SC_SLAB = 64;          // neurons per k_scores block = one mask word
constexpr int ROWS_THREADS = 512;    // k_rows block
constexpr int ROWS_WAVES = ROWS_THREADS / 64;
constexpr int ROWS_UB = 4;           // row kernels: rows of W_downT fetched together (the LDS row capacity is padded to this)
constexpr int SCAN_THREADS = 1024;   // k_compact_scan block
constexpr int ROWS_BLOCKS = 256;     // row-kernel blocks: one chunk of the row list and one partial y each (128 to
                                     // 512 were measured; 256 is best for every batch size)
constexpr int SC_TL = 4;             // k_scores: partials of t that a thread requests together
constexpr int SC_PG = 7;             // k_scores: sums of t read together
constexpr int RED_COLS = 8;          // k_reduce_y: float4 columns per block (one 128-byte line per partial row)
constexpr int RED_SEGS = 64;         // k_reduce_y: segments of the partial list per block

// Sum of a value over a block of 256 threads in a fixed order (the lanes of a wave, then the four waves); every thread gets it.
// The glue's sum of (x[j] + y[j])^2 ends here, in k_xP and in k_stack_glue.  What the threads bring is the same in both, so that the
// two give the same bits: a thread takes the 16-byte vectors t, t + 256, ... of x in ascending order, of each vector the elements in
// ascending order, with one fmaf(v, v, sum) each.  part: 4 floats of shared memory.
__device__ __forceinline__ float glue_block_total(float ss, float *part)
{
    const int tid = threadIdx.x;
    ss = wave_sum(ss);
    __syncthreads();
    if ((tid & 63) == 0) part[tid >> 6] = ss;
    __syncthreads();
    return ((part[0] + part[1]) + part[2]) + part[3];
}

// ---------------------------------------------------------------------------
// Predictor stage 1: partial t = x P over a tile of P   (Sec. 4.1 eq. 2: the
// inner factor B x of A B x + b, with P = B^T).
// Block (i, j) owns rows [i*XP_ROWS, +XP_ROWS) and columns [j*XP_COLS, +XP_COLS)
// of P [d][r] and writes tpart[i][b][its columns].  A thread owns one 16-byte
// column group and every NSUB-th row of the tile; its loads of P are issued
// while x is staged, and the NSUB row-partials are added through LDS in order.
// Dynamic LDS: NB*XP_ROWS + NSUB*(NB*XP_COLS + 1) + PARTS*NB*XP_COLS floats.
// ---------------------------------------------------------------------------
// With GLUE the token is not given but made here: x = RMSNorm(x_prev + y_prev) + shift rounded to
// the storage type, the stacked benchmark's glue (the order of the mean square's sum is k_stack_glue's,
// see glue_block_total, so the two give the same bits).  Every block forms the norm itself from the d sums of x_prev
// and y_prev (a few KB from L2) instead of waiting for one more launch; the blocks of the first
// column tile also write x to x_out for the row kernel.
// Bound: the trips.  Everything is asked for at the start, in the order of its use, so that the norm and x are there while P (from
// memory) is on its way; with P asked for first, every wait was for it, and the tile's own x and y came one trip after
// the sum.  With GLUE 5.05 -> 3.73 us at d = 4096, r = 256; eight stacked 7B layers 181.7 -> 172.0; without GLUE level.
template <typename W, int NB, bool GLUE>
__global__ __launch_bounds__(XP_THREADS) void k_xP(const W *__restrict__ P, const W *__restrict__ x,
                                                   int B, int d, int r, float *__restrict__ tpart,
                                                   const float *__restrict__ y_prev,
                                                   const float *__restrict__ shift, float eps,
                                                   W *__restrict__ x_out)
{
    constexpr int VEC = Elem<W>::VEC;
    constexpr int CG = XP_COLS / VEC;          // column groups per tile
    constexpr int NSUB = XP_THREADS / CG;      // row phases
    constexpr int RPT = XP_ROWS / NSUB;        // rows per thread
    extern __shared__ float smem[];
    float *xs = smem;                          // [NB][XP_ROWS]
    float *red = smem + NB * XP_ROWS;          // [NSUB][NB*XP_COLS + 1] (odd stride: no bank conflicts)
    const int tid = threadIdx.x;
    const int j0 = blockIdx.x * XP_ROWS;
    const int c0 = blockIdx.y * XP_COLS;
    const int cgi = tid % CG, sub = tid / CG;
    const int col = c0 + cgi * VEC;
    const bool colok = col < r;

    // ---- requested in the order in which they are used: what makes x, the tile's x, P ----
    const __amdgpu_buffer_rsrc_t tokens = range_of(x, (uint32_t)(B * d) * sizeof(W));
    const __amdgpu_buffer_rsrc_t before = range_of(y_prev, GLUE ? (uint32_t)(B * d) * 4 : 0u);
    constexpr int Y4 = VEC / 4;                // 16-byte vectors of y beside one of x
    constexpr int GV = 2;                      // vectors of a token's sum of squares under way per thread
    uint4 gx[GV], gy[GV][Y4];
    auto request_sum = [&](int b, int v0) {
#pragma unroll
        for (int k = 0; k < GV; ++k) {
            const int j = (v0 + tid + k * XP_THREADS) * VEC;
            gx[k] = load_range(tokens, j < d ? (uint32_t)(b * d + j) * sizeof(W) : OUTSIDE);
#pragma unroll
            for (int h = 0; h < Y4; ++h) gy[k][h] = load_range(before, j < d ? (uint32_t)(b * d + j + 4 * h) * 4u : OUTSIDE);
        }
    };
    if (GLUE) request_sum(0, 0);
    constexpr int XPT = XP_ROWS / VEC, XI = (NB * XPT + XP_THREADS - 1) / XP_THREADS;    // vectors of x: per token, per thread
    uint4 tx[XI], ty[XI][Y4], tsh[XI][Y4];
#pragma unroll
    for (int k = 0; k < XI; ++k) {
        const int i = tid + k * XP_THREADS, b = i / XPT, j = j0 + (i % XPT) * VEC;
        const bool in = b < B && j < d;
        tx[k] = load_range(tokens, in ? (uint32_t)(b * d + j) * sizeof(W) : OUTSIDE);
        if (GLUE) {
            const __amdgpu_buffer_rsrc_t shifts = range_of(shift, (uint32_t)d * 4);
#pragma unroll
            for (int h = 0; h < Y4; ++h) {
                ty[k][h] = load_range(before, in ? (uint32_t)(b * d + j + 4 * h) * 4u : OUTSIDE);
                tsh[k][h] = load_range(shifts, in ? (uint32_t)(j + 4 * h) * 4u : OUTSIDE);
            }
        }
    }
    uint4 raw[RPT];
    const __amdgpu_buffer_rsrc_t tile = range_of(P, (uint32_t)(d * r) * sizeof(W));
#pragma unroll
    for (int k = 0; k < RPT; ++k) {
        const int j = j0 + sub + k * NSUB;
        raw[k] = load_range(tile, colok && j < d ? (uint32_t)(j * r + col) * sizeof(W) : OUTSIDE);
    }
    __builtin_amdgcn_sched_barrier(0);

    __shared__ float gpart[4];
    float inv[NB];
    if (GLUE) {
        static_assert(XP_THREADS == 256, "a thread takes the vectors t, t + 256, ... of x, as in k_stack_glue");
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            inv[b] = 0.f;
            if (b == 0 || b < B) {             // B > 0: the first token's request stays where it is
                float ss = 0.f;
                auto add = [&] {
#pragma unroll
                    for (int k = 0; k < GV; ++k) {
                        float xv[VEC];
                        widen(gx[k], xv, (const W *)nullptr);
#pragma unroll
                        for (int h = 0; h < Y4; ++h) {
                            const float4 yv = as_float4(gy[k][h]);
                            const float a = xv[4 * h] + yv.x, bb = xv[4 * h + 1] + yv.y, c = xv[4 * h + 2] + yv.z,
                                        dd = xv[4 * h + 3] + yv.w;
                            ss = fmaf(a, a, ss);
                            ss = fmaf(bb, bb, ss);
                            ss = fmaf(c, c, ss);
                            ss = fmaf(dd, dd, ss);
                        }
                    }
                };
                if (b != 0) request_sum(b, 0);
                add();                         // apart from the loop: waits for its own loads only, not for P
                for (int v0 = GV * XP_THREADS; v0 * VEC < d; v0 += GV * XP_THREADS) {
                    request_sum(b, v0);
                    add();
                }
                inv[b] = 1.0f / sqrtf(glue_block_total(ss, gpart) / (float)d + eps);
            }
        }
    }
#pragma unroll
    for (int k = 0; k < XI; ++k) {
        const int i = tid + k * XP_THREADS, b = i / XPT, j = j0 + (i % XPT) * VEC;
        if (i >= NB * XPT) break;
        float w[VEC];
        widen(tx[k], w, (const W *)nullptr);
        if (GLUE && b < B && j < d) {
            float f = inv[0];
#pragma unroll
            for (int q = 1; q < NB; ++q) f = b == q ? inv[q] : f;
            W rounded[VEC];
#pragma unroll
            for (int h = 0; h < Y4; ++h) {
                const float4 yv = as_float4(ty[k][h]), sv = as_float4(tsh[k][h]);
                const float add[4] = {yv.x, yv.y, yv.z, yv.w}, sh[4] = {sv.x, sv.y, sv.z, sv.w};
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float v = (w[4 * h + e] + add[e]) * f + sh[e];
                    from_f32(v, &rounded[4 * h + e]);
                    w[4 * h + e] = to_f32(rounded[4 * h + e]);
                }
            }
            if (blockIdx.y == 0) {
#pragma unroll
                for (int e = 0; e < VEC; ++e) x_out[(size_t)b * d + j + e] = rounded[e];
            }
        }
#pragma unroll
        for (int e = 0; e < VEC; ++e) xs[b * XP_ROWS + (j - j0) + e] = w[e];
    }
    __syncthreads();

    float acc[NB][VEC];
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int e = 0; e < VEC; ++e) acc[b][e] = 0.f;
#pragma unroll
    for (int k = 0; k < RPT; ++k) {
        const int jj = sub + k * NSUB;
        if (colok && j0 + jj < d) {
            float w[VEC];
            widen(raw[k], w, (const W *)nullptr);
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                const float xv = xs[b * XP_ROWS + jj];
#pragma unroll
                for (int e = 0; e < VEC; ++e) acc[b][e] = fmaf(xv, w[e], acc[b][e]);
            }
        }
    }
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int e = 0; e < VEC; ++e) red[sub * (NB * XP_COLS + 1) + b * XP_COLS + cgi * VEC + e] = acc[b][e];
    __syncthreads();
    // two-level sum of the NSUB row phases (fixed order): the NB*XP_COLS outputs of the
    // tile are shared out over the block, PARTS threads per output
    constexpr int OUTS = NB * XP_COLS;
    constexpr int PARTS = XP_THREADS / OUTS >= 1 ? XP_THREADS / OUTS : 1;
    constexpr int PER = NSUB / PARTS;
    float *red2 = red + NSUB * (OUTS + 1);                   // [PARTS][OUTS]
    for (int o = tid % OUTS, part = tid / OUTS; part < PARTS; part += XP_THREADS) {
        float s = 0.f;
#pragma unroll 8
        for (int q = 0; q < PER; ++q) s += red[(part * PER + q) * (OUTS + 1) + o];
        red2[part * OUTS + o] = s;
    }
    __syncthreads();
    for (int o = tid; o < OUTS; o += XP_THREADS) {
        const int b = o / XP_COLS, k = o % XP_COLS;
        if (c0 + k < r) {
            float t = 0.f;
#pragma unroll
            for (int q = 0; q < PARTS; ++q) t += red2[q * OUTS + o];
            tpart[((size_t)blockIdx.x * NB + b) * r + c0 + k] = t;
        }
    }
}

// ---------------------------------------------------------------------------
// Sum of the nt stage-1 partials into one t (fixed order).  Used by the vector engine for batches of
// three or more tokens, where re-adding the partials in every score block would
// cost more than this extra launch.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_tsum(const float *__restrict__ tpart, int nt, int count,
                                              float *__restrict__ t)
{
    const int c = blockIdx.x * 256 + threadIdx.x;
    if (c >= count) return;
    float s = 0.f;
#pragma unroll 8
    for (int g = 0; g < nt; ++g) s += tpart[(size_t)g * count + c];
    t[c] = s;
}

// ---------------------------------------------------------------------------
// Predictor stage 2 + step function: s_i = t . Q[i,:] + b_i for one slab of 64
// neurons, then (optionally) the 64-bit mask word of the slab:
// bit j = OR over tokens of [s > 0]   (eq. 2's H; the union over the batch).
// A group of LPR = 2^LPR_LOG2 lanes owns every NGRP-th row of the slab; a lane
// owns the column groups lig, lig+LPR, ... of its rows.
// Bound: one trip to memory and the hand-overs behind it.  The nt stage-1 partials of t are requested first (npg threads per
// column share them, SC_TL at a time and thread), then the rows' first column groups, so that t is put together (fixed order,
// through LDS) while Q is on its way; the first SC_TL are added outside of the loop over further ones, because a wait inside
// of it would be for Q as well.  7B step 18.1 -> 16.8 us with this and k_reduce_y's loads together, eight stacked layers 199.8 ->
// 190.0 (loops of one load and one add each, two trips here and up to four there; sums in LDS read one by one).
// SC_THREADS is 512 for one or two tokens (short critical path) and 256 for larger
// batches (fewer wavefronts repeating the per-wave overhead).
// Dynamic LDS: NB*r + NB*64 + max(SC_THREADS*4, NB*r) floats.
// ---------------------------------------------------------------------------
template <typename W, int NB, int LPR_LOG2, int SC_THREADS>
__global__ __launch_bounds__(SC_THREADS) __attribute__((amdgpu_waves_per_eu(2, 4))) void k_scores(const W *__restrict__ Q,
                                                       const float *__restrict__ bias,
                                                       const float *__restrict__ tpart, int nt, int npg, int r, int B,
                                                       uint64_t *__restrict__ mask_out, float *__restrict__ s_out, int D)
{
    constexpr int VEC = Elem<W>::VEC;
    constexpr int LPR = 1 << LPR_LOG2;              // lanes per row: 8, 16, 32 or 64
    constexpr int NGRP = SC_THREADS / LPR;          // lane groups per block
    constexpr int RPG = (SC_SLAB + NGRP - 1) / NGRP;   // rows per lane group (groups beyond the slab idle)
    extern __shared__ float smem[];
    float *ts = smem;                  // [NB][r]
    float *sc = ts + NB * r;           // [NB][64]
    float *tsp = sc + NB * SC_SLAB;    // [npg][NB*r] partial sums of t
    const int tid = threadIdx.x;
    const int i0 = blockIdx.x * SC_SLAB;
    const int lig = tid & (LPR - 1);
    const int grp = tid >> LPR_LOG2;
    const int cg = r / VEC;

    // t: thread (pg, cq) adds the partials pg, pg + npg, ... of its float4 column; npg > 1 only where one pass has room for all
    const int ncq = NB * r / 4;
    const __amdgpu_buffer_rsrc_t parts = range_of(tpart, (uint32_t)nt * ncq * 16);
    uint4 tq[SC_TL];
    int pg = 0, cq = tid;
    if (npg > 1) {                     // tid / ncq, tid < 512
        pg = (int)(((float)tid + 0.5f) * __builtin_amdgcn_rcpf((float)ncq));
        cq = tid - pg * ncq;
    }
    auto request_t = [&](int k0) {
#pragma unroll
        for (int k = 0; k < SC_TL; ++k)
            tq[k] = load_range(parts, pg < npg && cq < ncq ? (uint32_t)((pg + (k0 + k) * npg) * ncq + cq) * 16u : OUTSIDE);
    };
    auto add_t = [&](float4 s) {
#pragma unroll
        for (int k = 0; k < SC_TL; ++k) {
            const float4 p = as_float4(tq[k]);
            s.x += p.x; s.y += p.y; s.z += p.z; s.w += p.w;
        }
        return s;
    };
    request_t(0);

    // first column group of each of this group's rows, and the bias (added after the row sums)
    uint4 raw[RPG];
    const bool has_rows = NGRP <= SC_SLAB || grp < SC_SLAB;
    const W *qrow = Q + (size_t)(i0 + (has_rows ? grp : 0)) * r + (lig < cg ? lig : 0) * VEC;
#pragma unroll
    for (int k = 0; k < RPG; ++k) raw[k] = load_raw(qrow + (size_t)k * NGRP * r);
    const float my_bias = bias[i0 + (tid & (SC_SLAB - 1))];
    __builtin_amdgcn_sched_barrier(0);

    {   // t = sum of the stage-1 partials
        float4 *tsp4 = reinterpret_cast<float4 *>(tsp);
        auto finish_t = [&](float4 s) {
            for (int k0 = SC_TL; k0 * npg < nt; k0 += SC_TL) {
                request_t(k0);
                s = add_t(s);
            }
            if (pg < npg && cq < ncq) tsp4[pg * ncq + cq] = s;
        };
        finish_t(add_t(make_float4(0.f, 0.f, 0.f, 0.f)));          // apart from the loop: waits for its own loads only
        if (npg == 1) {
            for (int c0 = SC_THREADS; c0 < ncq; c0 += SC_THREADS) {
                cq = c0 + tid;
                request_t(0);
                finish_t(add_t(make_float4(0.f, 0.f, 0.f, 0.f)));
            }
        }
        __syncthreads();
        float4 *ts4 = reinterpret_cast<float4 *>(ts);
        for (int c = tid; c < ncq; c += SC_THREADS) {
            float4 s = tsp4[c];
            for (int q0 = 1; q0 < npg; q0 += SC_PG) {
                float4 p[SC_PG];
#pragma unroll
                for (int k = 0; k < SC_PG; ++k) p[k] = tsp4[min(q0 + k, npg - 1) * ncq + c];
#pragma unroll
                for (int k = 0; k < SC_PG; ++k) {
                    const bool in = q0 + k < npg;
                    s.x += in ? p[k].x : 0.f; s.y += in ? p[k].y : 0.f; s.z += in ? p[k].z : 0.f; s.w += in ? p[k].w : 0.f;
                }
            }
            ts4[c] = s;
        }
        __syncthreads();
    }

    float acc[RPG][NB];
#pragma unroll
    for (int k = 0; k < RPG; ++k)
#pragma unroll
        for (int b = 0; b < NB; ++b) acc[k][b] = 0.f;
    if (lig < cg) {
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            float tv[VEC];
#pragma unroll
            for (int e = 0; e < VEC; ++e) tv[e] = ts[b * r + lig * VEC + e];
#pragma unroll
            for (int k = 0; k < RPG; ++k) {
                float w[VEC];
                widen(raw[k], w, (const W *)nullptr);
#pragma unroll
                for (int e = 0; e < VEC; ++e) acc[k][b] = fmaf(tv[e], w[e], acc[k][b]);
            }
        }
    }
    for (int v = lig + LPR; v < cg && has_rows; v += LPR) {          // only when r/VEC > 64
        for (int k = 0; k < RPG; ++k) {
            float w[VEC];
            load_vec(Q + (size_t)(i0 + grp + k * NGRP) * r + v * VEC, w);
#pragma unroll
            for (int b = 0; b < NB; ++b)
#pragma unroll
                for (int e = 0; e < VEC; ++e) acc[k][b] = fmaf(ts[b * r + v * VEC + e], w[e], acc[k][b]);
        }
    }
#pragma unroll
    for (int k = 0; k < RPG; ++k)
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            const float t = group_sum<LPR_LOG2>(acc[k][b]);
            if (lig == 0 && has_rows) sc[b * SC_SLAB + grp + k * NGRP] = t;
        }
    __syncthreads();
    if (tid < SC_SLAB) {
        bool on = false;
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            const float v = sc[b * SC_SLAB + tid] + my_bias;
            if (b < B) {
                on = on || v > 0.f;
                if (s_out != nullptr) s_out[(size_t)b * D + i0 + tid] = v;
            }
        }
        const uint64_t m = __ballot(on);
        if (mask_out != nullptr && tid == 0) mask_out[blockIdx.x] = m;
    }
}

// ---------------------------------------------------------------------------
// Mask words from materialised scores: one wave per word, bit j of word k is
// neuron 64k + j, set iff s[t][64k+j] > 0 for some token t.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_mask_from_scores(const float *__restrict__ s, int B, int D,
                                                          uint64_t *__restrict__ mask)
{
    const int lane = threadIdx.x & 63;
    const int k = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (k >= D / 64) return;
    bool on = false;
    for (int b = 0; b < B; ++b) on = on || (s[(size_t)b * D + (size_t)k * 64 + lane] > 0.f);
    const uint64_t m = __ballot(on);
    if (lane == 0) mask[k] = m;
}

// ---------------------------------------------------------------------------
// Mask words -> ascending index list and its length (Alg. 4's nonzero).
// One block: popcount per word, block-wide exclusive scan (wave scan +
// 16 wave totals), then one wave per word writes its set bits at
// offset[word] + (number of set bits below the lane).
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(SCAN_THREADS) void k_compact_scan(const uint64_t *__restrict__ mask,
                                                               int nwords, int32_t *__restrict__ idx,
                                                               int32_t *__restrict__ nnz)
{
    __shared__ int wsum[SCAN_THREADS / 64];
    __shared__ int offs[SCAN_THREADS];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    int running = 0;
    for (int base = 0; base < nwords; base += SCAN_THREADS) {
        const int k = base + tid;
        const uint64_t w = k < nwords ? mask[k] : 0ull;
        const int c = __popcll(w);
        const int inc = wave_inclusive_scan(c);
        if (lane == 63) wsum[wave] = inc;
        __syncthreads();
        int wbase = 0, tot = 0;
        for (int q = 0; q < SCAN_THREADS / 64; ++q) {
            const int s = wsum[q];
            if (q < wave) wbase += s;
            tot += s;
        }
        offs[tid] = running + wbase + inc - c;
        __syncthreads();
        const int nw_here = min(SCAN_THREADS, nwords - base);
        for (int kk = wave; kk < nw_here; kk += SCAN_THREADS / 64) {
            const uint64_t ww = mask[base + kk];
            if ((ww >> lane) & 1ull) {
                const int below = __popcll(ww & ((1ull << lane) - 1ull));
                idx[offs[kk] + below] = (base + kk) * 64 + lane;
            }
        }
        running += tot;
        __syncthreads();
    }
    if (tid == 0) *nnz = running;
}

// ---------------------------------------------------------------------------
// Gate, up and down over a list of rows (Alg. 3's SparseGate / SparseUpAndMul /
// SparseDown in one launch).  Where the list comes from:
//   ROWS_DENSE : all D rows (eq. 1, the dense baseline)
//   ROWS_LIST  : idx_in[0 .. *nnz_in)           (svdp_sparse_ffn)
//   ROWS_MASK  : the set bits of mask[0 .. D/64) (svdp_ffn_step): every block
//                scans the popcounts of the mask words itself (Alg. 4's
//                nonzero, without a separate launch) and extracts its own
//                part of the ascending list; when idx_out / nnz_out are given
//                each block also writes its part of the list there.
// `list` is idx_in or mask; dB = d | B << 16 (arguments beyond the first fourteen words are not there at the start).
// The list of n rows is cut into gridDim.x contiguous chunks; block g handles
// chunk g:
//   phase A: one wave per row: g = W_gate[i].x, u = W_up[i].x (wave reduction),
//            h = ReLU(g)*u to LDS;
//   phase B: every thread owns 16-byte column groups of the output and adds
//            h * W_downT[i][cols] over the chunk in list order -> ypart[g].
//            The first rows of W_downT are requested before phase A starts.
// Blocks with an empty chunk write no partial y; block 0 records n and the number of partials for k_reduce_y.
// The LDS row capacity is a multiple of ROWS_UB.
// Dynamic LDS: NB*d storage elements (x as stored), NB*max_chunk floats, max_chunk ints, up to all of a compute unit's: no static LDS.
// ---------------------------------------------------------------------------
enum RowsMode { ROWS_DENSE = 0, ROWS_LIST = 1, ROWS_MASK = 2 };

// Rows per block: the list of n rows is cut into contiguous chunks of
// max(min_chunk, ceil(n / G)) rows, so that a short list occupies fewer blocks and leaves
// fewer partial y's to write and sum.  (Spreading a list of ~1000 rows of the 7B shape over every
// compute unit is 0.3 us faster in the row kernel than four rows per block and 1.3 us faster than
// eight, measured; four costs the step nothing, because the sum of the partials gains what the
// row kernel loses, and halves the partial-y traffic of short lists.)
__device__ __forceinline__ int chunk_of(int n, int G, int min_chunk) { return max(min_chunk, (n + G - 1) / G); }
constexpr int ROWS_MIN_CHUNK = 4;   // of k_rows and k_rows_seq
// LDS row capacity of a block of a row kernel: its share of all D rows, in whole groups.
__host__ __device__ constexpr int rows_max_chunk(int D, int min_chunk, int group)
{
    const int per = (D + ROWS_BLOCKS - 1) / ROWS_BLOCKS, most = per > min_chunk ? per : min_chunk;
    return (most + group - 1) / group * group;
}
// Blocks that get rows (= partial y's written).
__device__ __forceinline__ int active_blocks(int n, int chunk) { return n > 0 ? (n + chunk - 1) / chunk : 0; }

// Length n of the row list.  ROWS_MASK: every wave scans the popcounts of all mask words
// by itself (lane l owns the wpl consecutive words starting at l*wpl), so no block-wide
// step is needed; lane_first is the list position of the lane's first set bit.  The
// lane's first ROWS_WREG words stay in registers (held[]) for rows_list_from_mask.
constexpr int ROWS_WREG = 8;        // covers D <= 32768; the second half is only asked for where D > 16384
template <int MODE>
__device__ __forceinline__ void rows_request_mask(int D, const void *__restrict__ list, int lane, int &wpl,
                                                  uint64_t (&held)[ROWS_WREG])
{
    const int nwords = D / 64;
    wpl = (nwords + 63) / 64;
#pragma unroll
    for (int j = 0; j < ROWS_WREG; ++j) held[j] = 0ull;
    if (MODE != ROWS_MASK) return;
    const __amdgpu_buffer_rsrc_t words = range_of(list, (uint32_t)nwords * 8);
#pragma unroll
    for (int j = 0; j < ROWS_WREG / 2; ++j) held[j] = load_range_8(words, j < wpl ? (uint32_t)(lane * wpl + j) * 8u : OUTSIDE);
    if (wpl > ROWS_WREG / 2) {
#pragma unroll
        for (int j = ROWS_WREG / 2; j < ROWS_WREG; ++j)
            held[j] = load_range_8(words, j < wpl ? (uint32_t)(lane * wpl + j) * 8u : OUTSIDE);
    }
}
template <int MODE>
__device__ __forceinline__ int rows_list_length(int D, const void *__restrict__ list, const int32_t *__restrict__ nnz_in,
                                                int lane, int wpl, const uint64_t (&held)[ROWS_WREG], int &lane_first)
{
    lane_first = 0;
    if (MODE == ROWS_DENSE) return D;
    if (MODE == ROWS_LIST) return max(0, min(*nnz_in, D));
    int c = 0;
#pragma unroll
    for (int j = 0; j < ROWS_WREG; ++j) c += __popcll(held[j]);
    for (int j = ROWS_WREG; j < wpl; ++j) {
        const int k = lane * wpl + j;
        if (k < D / 64) c += __popcll(static_cast<const uint64_t *>(list)[k]);
    }
    const int inc = wave_inclusive_scan(c);
    lane_first = inc - c;
    return __builtin_amdgcn_readlane(inc, 63);
}

// Entries [lo, hi) of the ascending list of set mask bits -> lidx[0 .. hi-lo), by one wave.
// Lane l knows where its words start in the list (lane_first).  Words that overlap
// [lo, hi) are handed to the whole wave one at a time: lane j then looks at bit j, whose
// list position is the word's start plus the number of set bits below it.
__device__ __forceinline__ void rows_list_word(uint64_t w, int j, int wpl, int lane, int &p, int lo, int hi, int *lidx)
{
    const int pc = __popcll(w);
    const bool overlaps = pc > 0 && p < hi && p + pc > lo;
    uint64_t todo = __ballot(overlaps);
    while (todo != 0ull) {
        const int src = __ffsll((unsigned long long)todo) - 1;
        todo &= todo - 1ull;
        const uint32_t wlo = __builtin_amdgcn_readlane((uint32_t)w, src);
        const uint32_t whi = __builtin_amdgcn_readlane((uint32_t)(w >> 32), src);
        const int pk = __builtin_amdgcn_readlane(p, src);
        const uint64_t wk = ((uint64_t)whi << 32) | wlo;
        if ((wk >> lane) & 1ull) {
            const int pos = pk + __popcll(wk & ((1ull << lane) - 1ull));
            if (pos >= lo && pos < hi) lidx[pos - lo] = (src * wpl + j) * 64 + lane;
        }
    }
    p += pc;
}
__device__ __forceinline__ void rows_list_from_mask(int D, const void *__restrict__ list, int lane,
                                                    int lane_first, int wpl, const uint64_t (&held)[ROWS_WREG], int lo,
                                                    int hi, int *lidx)
{
    const int nwords = D / 64;
    int p = lane_first;
#pragma unroll
    for (int j = 0; j < ROWS_WREG; ++j)
        if (j < wpl) rows_list_word(held[j], j, wpl, lane, p, lo, hi, lidx);
    for (int j = ROWS_WREG; j < wpl; ++j) {
        const int k = lane * wpl + j;
        rows_list_word(k < nwords ? static_cast<const uint64_t *>(list)[k] : 0ull, j, wpl, lane, p, lo, hi, lidx);
    }
}

// This block's part of the row list into lidx[0 .. cnt): from the caller's list (entries outside
// [0, D) become -1 and are skipped by every row kernel: they contribute nothing), from the mask
// words (wave 0), or the block's own range of all rows.  Ends with a block barrier.
template <int MODE>
__device__ __forceinline__ void rows_block_list(int D, const void *__restrict__ list, int lane_first, int wpl,
                                                const uint64_t (&held)[ROWS_WREG], int lo, int hi, int *lidx)
{
    const int tid = threadIdx.x, cnt = hi - lo;
    if (MODE == ROWS_LIST) {
        for (int q = tid; q < cnt; q += blockDim.x) {
            const int i = static_cast<const int32_t *>(list)[lo + q];
            lidx[q] = (unsigned)i < (unsigned)D ? i : -1;
        }
    } else if (MODE == ROWS_MASK) {
        if (tid < 64) rows_list_from_mask(D, list, tid, lane_first, wpl, held, lo, hi, lidx);
    } else {
        for (int q = tid; q < cnt; q += blockDim.x) lidx[q] = lo + q;
    }
    __syncthreads();
}

// Whether the rows of a list are read past the caches: from 64 MB on with one or two tokens, from 100 MB on with more.  Gains where the
// weights come from memory, as in a model of many layers, loses where one layer's are called again and again and fit the memory-side
// cache.  Read as usual -> past the caches, us, from memory (1.5 GB of listed rows in turn) / the same layer: k_rows, d = 2560, one token,
// 64 MB 18.2 -> 16.7, 144 MB 30.4 -> 28.0 / 25.4 -> 25.6, 256 MB 48.5 -> 44.0; d = 4096, two tokens, 80 MB 22.1 -> 21.7 / 19.1 -> 19.9, 144 MB 31.5 ->
// 29.9 / 26.6 -> 28.2; four tokens, 64 MB 23.0 -> 24.1, 80 MB 26.4 -> 26.4 / 23.3 -> 26.1, 112 MB 30.8 -> 30.4 / 27.0 -> 30.4, 144 MB 36.0 -> 34.2 /
// 30.5 -> 34.2, 256 MB 54.9 -> 50.4, 320 MB 65.8 -> 59.4.  What they leave in the caches is the predictor: whole step, four tokens, 105 MB
// of 4096 x 14336 38.2 -> 36.1 / 33.7 -> 36.2, 134 MB of 3584 x 18944 48.1 -> 45.8 / 43.0 -> 45.2.
// k_down_slices, both row kernels of eight tokens: d = 4096, 48 MB 22.4 -> 22.4, 112 MB 34.6 -> 34.1 / 30.8 -> 31.9, 200 MB 47.7 -> 47.0, 320 MB 71.7 ->
// 69.8; d = 2560, 144 MB 43.2 -> 42.7.  k_gate_up_mfma always reads as usual, since it fetches a line in two halves: the same two, past the caches
// in both, 25.1, 35.3, 49.3 and 73.5 (only the first pass after a layer's weights have been written gains from it: step of 4096 x 14336, eight
// tokens 98 -> 83, later ones 64 -> 69: what is read as usual has to wait for written lines to leave the caches).  k_rows_seq as well: not measured otherwise.
__device__ __forceinline__ bool streams(int tokens, int n, int d, int bytes)
{
    return (float)n * (float)(3 * d * bytes) >= (tokens <= 2 ? 64e6f : 100e6f);
}

// x [B][d] as stored into xraw [NB][nvec] (zeros beyond B), in two halves: the first XV vectors of a thread are
// requested behind whatever the caller asked for before and stored once that has been used; rows longer than that follow in a loop.
constexpr int ROWS_XV = 2;
template <typename W, int NB, int XV>
__device__ __forceinline__ void rows_request_x(const W *__restrict__ x, int B, int d, int v0, uint4 (&xv)[XV][NB])
{
    constexpr int VEC = Elem<W>::VEC;
    const __amdgpu_buffer_rsrc_t tokens = range_of(x, (uint32_t)(B * d) * sizeof(W));
#pragma unroll
    for (int k = 0; k < XV; ++k)
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            const int v = v0 + threadIdx.x + k * ROWS_THREADS;
            xv[k][b] = load_range(tokens, v * VEC < d ? (uint32_t)(b * d + v * VEC) * sizeof(W) : OUTSIDE);
        }
}

// Bound: for a short list, the trips: mask and x, the rows, the partial outputs' way out; for a long one the stream.  So each phase
// asks for everything it will need before it waits: the first rows of W_downT before phase A, a row's vectors of both
// matrices at once and the next row's before this one's sums are taken, two groups of W_downT rows in turn.  (The requests stand outside
// of branches, as ranges that end where the row does: a branch there made the compiler wait for each.)
// Against loads in branches, two of them waited for one by one and the rest of a row in two trips: dense FFN of 5120 x 13824
// 82.0 -> 76.7 us, step of 3584 x 18944, four tokens (33 % of the rows) 54.9 -> 51.6, ragged list of 1507 rows 12.4 -> 11.9, eight
// stacked 7B layers 190.0 -> 183.
template <typename W, int NB, int MODE>
__global__ __launch_bounds__(ROWS_THREADS) __attribute__((amdgpu_waves_per_eu(2, 4))) void k_rows(
    const W *__restrict__ x, const void *__restrict__ list, const W *__restrict__ Wg, const W *__restrict__ Wu,
    const W *__restrict__ WdT, const int32_t *__restrict__ nnz_in, int dB, int D, uint32_t flags, int32_t *__restrict__ idx_out,
    int32_t *__restrict__ nnz_out, int32_t *__restrict__ n_used, float *__restrict__ ypart)
{
    constexpr int VEC = Elem<W>::VEC;
    constexpr int UA = 8;                   // 16-byte loads in flight per matrix in phase A
    constexpr int UB = ROWS_UB;             // rows of W_downT per group in phase B
    extern __shared__ uint4 smem16[];
    const int d = dB & 0xffff, B = NB == 1 ? 1 : dB >> 16;
    const int nvec = d / VEC, max_chunk = rows_max_chunk(D, ROWS_MIN_CHUNK, UB);
    uint4 *xraw = smem16;                                        // [NB][nvec] x in storage form
    float *hs = reinterpret_cast<float *>(xraw + NB * nvec);     // [NB][max_chunk]
    int *lidx = reinterpret_cast<int *>(hs + NB * max_chunk);    // [max_chunk]
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    // ---- request the mask words, then x ----
    int lane_first, wpl;
    uint64_t held[ROWS_WREG];
    rows_request_mask<MODE>(D, list, lane, wpl, held);
    uint4 xv[ROWS_XV][NB];
    rows_request_x<W, NB>(x, B, d, 0, xv);

    // ---- the list: n, this block's chunk [lo, hi) ----
    const int n = rows_list_length<MODE>(D, list, nnz_in, lane, wpl, held, lane_first);
    const int chunk = chunk_of(n, ROWS_BLOCKS, ROWS_MIN_CHUNK);
    const int lo = min(n, (int)blockIdx.x * chunk);
    const int hi = min(n, lo + chunk);
    const int cnt = hi - lo;
    // written at the kernel's end: a wait for loads waits for the stores in front of them too
    auto store_list = [&] {
        if (blockIdx.x == 0 && tid == 0) {
            if (MODE != ROWS_DENSE) *reinterpret_cast<int2 *>(n_used) = make_int2(n, active_blocks(n, chunk));
            if (MODE == ROWS_MASK && nnz_out != nullptr) *nnz_out = n;
        }
        if (MODE == ROWS_MASK && idx_out != nullptr)
            for (int q = tid; q < cnt; q += ROWS_THREADS) idx_out[lo + q] = lidx[q];
    };
    if (cnt <= 0) {
        store_list();
        return;
    }

    for (int v0 = 0; v0 < nvec; v0 += ROWS_XV * ROWS_THREADS) {
        if (v0 != 0) rows_request_x<W, NB>(x, B, d, v0, xv);
#pragma unroll
        for (int k = 0; k < ROWS_XV; ++k)
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                const int v = v0 + tid + k * ROWS_THREADS;
                if (v < nvec) xraw[b * nvec + v] = xv[k][b];
            }
    }
    // h of the positions past the chunk's end (phase B works in whole groups of UB rows)
    const int ngroups = (cnt + UB - 1) / UB;
    if (tid < ngroups * UB - cnt) {
#pragma unroll
        for (int b = 0; b < NB; ++b) hs[b * max_chunk + cnt + tid] = 0.f;
    }
    rows_block_list<MODE>(D, list, lane_first, wpl, held, lo, hi, lidx);

    const bool drelu = (flags & 1u) != 0;
    const uint32_t row_bytes = (uint32_t)d * sizeof(W);
    // row i of a matrix; nothing at all where i < 0 (past the end; a rejected entry of the caller's list)
    auto row_range = [&](const W *M, int i) { return range_of(M + (size_t)max(i, 0) * d, i >= 0 ? row_bytes : 0u); };
    auto work = [&](auto stream, auto ragged) {
        constexpr bool STREAM = decltype(stream)::value, RAGGED = decltype(ragged)::value;
        // rows UB g .. UB g + UB - 1 of the chunk, at byte `at` of each; zeros past the end
        auto fetch = [&](int g, uint32_t at, uint4 (&piece)[UB]) {
            static_assert(UB == 4, "one 16-byte read of the list");
            int row[UB];
            if (MODE == ROWS_DENSE) {
#pragma unroll
                for (int k = 0; k < UB; ++k) row[k] = lo + g * UB + k;
            } else {
                const int4 r4 = *reinterpret_cast<const int4 *>(lidx + min(g, ngroups - 1) * UB);
                row[0] = __builtin_amdgcn_readfirstlane(r4.x);
                row[1] = __builtin_amdgcn_readfirstlane(r4.y);
                row[2] = __builtin_amdgcn_readfirstlane(r4.z);
                row[3] = __builtin_amdgcn_readfirstlane(r4.w);
            }
#pragma unroll
            for (int k = 0; k < UB; ++k) piece[k] = load_range<STREAM>(row_range(WdT, g * UB + k < cnt ? row[k] : -1), at);
        };
        // ---- request the first group of W_downT rows for this thread's first column group ----
        uint4 pa[UB], pb[UB];
        fetch(0, (uint32_t)tid * 16u, pa);

        // ---- phase A: one wave per row, 64 UA vectors of both matrices at a time ----
        uint4 rg[UA], ru[UA];
        auto request = [&](int q, int vb) {
            const int row = __builtin_amdgcn_readfirstlane(MODE == ROWS_DENSE ? lo + q : lidx[q]);
            const __amdgpu_buffer_rsrc_t g = row_range(Wg, row), u = row_range(Wu, row);
            const uint32_t at = (uint32_t)(vb + lane) * 16u;
#pragma unroll
            for (int k = 0; k < UA / 2; ++k) {
                rg[k] = load_range<STREAM>(g, at + k * 1024);
                ru[k] = load_range<STREAM>(u, at + k * 1024);
            }
            if (vb + UA / 2 * 64 < nvec) {
#pragma unroll
                for (int k = UA / 2; k < UA; ++k) {
                    rg[k] = load_range<STREAM>(g, at + k * 1024);
                    ru[k] = load_range<STREAM>(u, at + k * 1024);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        };
        if (wave < cnt) request(wave, 0);
        float ag[NB], au[NB];
#pragma unroll
        for (int b = 0; b < NB; ++b) ag[b] = au[b] = 0.f;
        for (int q = wave, vb = 0; q < cnt;) {
            // Lanes past the row's end take no part: their weights of zero would make NaN of an infinite x.  One and two tokens: halves that
            // lie in the row as a whole have no test, in the others x is read in front of it (a read behind each test is awaited by
            // itself).  Against x cleared in every product (one token) or a test around each (two): eight stacked 7B layers 178.5 ->
            // 177.5 us, list of 1507 rows of 2824 12.09 -> 12.02, dense 5120 x 13824 68.9 -> 69.0.  More tokens: the products are
            // longer than the reads; the split as above 47.6 -> 48.0 (3584 x 18944, four tokens).
            auto half = [&](int k0) {
                auto product = [&](int k, int b, const uint4 &xq) {
                    ag[b] = dot_raw(rg[k], xq, ag[b], (const W *)nullptr);
                    au[b] = dot_raw(ru[k], xq, au[b], (const W *)nullptr);
                };
                const int v0 = vb + k0 * 64 + lane;
                if (!RAGGED || (NB <= 2 && vb + (k0 + UA / 2) * 64 <= nvec)) {
#pragma unroll
                    for (int k = 0; k < UA / 2; ++k)
#pragma unroll
                        for (int b = 0; b < NB; ++b) product(k0 + k, b, xraw[b * nvec + v0 + k * 64]);
                } else if (NB <= 2) {
                    uint4 xq[UA / 2][NB];
#pragma unroll
                    for (int k = 0; k < UA / 2; ++k)
#pragma unroll
                        for (int b = 0; b < NB; ++b) xq[k][b] = xraw[b * nvec + min(v0 + k * 64, nvec - 1)];
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int k = 0; k < UA / 2; ++k)
                        if (v0 + k * 64 < nvec) {
#pragma unroll
                            for (int b = 0; b < NB; ++b) product(k0 + k, b, xq[k][b]);
                        }
                } else {
#pragma unroll
                    for (int k = 0; k < UA / 2; ++k)
                        if (v0 + k * 64 < nvec) {
#pragma unroll
                            for (int b = 0; b < NB; ++b) product(k0 + k, b, xraw[b * nvec + v0 + k * 64]);
                        }
                }
            };
            half(0);
            if (vb + UA / 2 * 64 < nvec) half(UA / 2);
            const bool whole = vb + UA * 64 >= nvec;                     // the row is done
            const int nq = whole ? q + ROWS_WAVES : q, nvb = whole ? 0 : vb + UA * 64;
            if (nq < cnt) request(nq, nvb);
            if (whole) {
                const bool valid = MODE != ROWS_LIST || lidx[q] >= 0;
#pragma unroll
                for (int b = 0; b < NB; ++b) {
                    const float gs = wave_sum(ag[b]);
                    const float us = wave_sum(au[b]);
                    if (lane == 0) {
                        const float gp = fmaxf(gs, 0.f);
                        const float uu = drelu ? fmaxf(us, 0.f) : us;
                        hs[b * max_chunk + q] = valid ? gp * uu : 0.f;
                    }
                    ag[b] = au[b] = 0.f;
                }
            }
            q = nq;
            vb = nvb;
        }
        __syncthreads();

        // ---- phase B: every thread owns 16-byte column groups of the output ----
        for (int v = tid; v < nvec; v += ROWS_THREADS) {
            float acc[NB][VEC];
#pragma unroll
            for (int b = 0; b < NB; ++b)
#pragma unroll
                for (int e = 0; e < VEC; ++e) acc[b][e] = 0.f;
            const uint32_t at = (uint32_t)v * 16u;
            auto add = [&](int g, const uint4 (&piece)[UB]) {
                float h[NB][UB];
#pragma unroll
                for (int b = 0; b < NB; ++b) {
                    const float4 h4 = *reinterpret_cast<const float4 *>(hs + b * max_chunk + min(g, ngroups - 1) * UB);
                    const bool in = g < ngroups;
                    h[b][0] = in ? h4.x : 0.f; h[b][1] = in ? h4.y : 0.f; h[b][2] = in ? h4.z : 0.f; h[b][3] = in ? h4.w : 0.f;
                }
#pragma unroll
                for (int k = 0; k < UB; ++k) {
                    float w[VEC];
                    widen(piece[k], w, (const W *)nullptr);
#pragma unroll
                    for (int b = 0; b < NB; ++b)
#pragma unroll
                        for (int e = 0; e < VEC; ++e) acc[b][e] = fmaf(h[b][k], w[e], acc[b][e]);
                }
            };
            if (v != tid) fetch(0, at, pa);
            if (ngroups == 1) {
                add(0, pa);
            } else {
                for (int g = 0; g < ngroups; g += 2) {          // a group past the end adds zeros: a test would draw its loads in
                    fetch(g + 1, at, pb);
                    __builtin_amdgcn_sched_barrier(0);
                    add(g, pa);
                    fetch(g + 2, at, pa);
                    __builtin_amdgcn_sched_barrier(0);
                    add(g + 1, pb);
                }
            }
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                float4 *out = reinterpret_cast<float4 *>(ypart + ((size_t)blockIdx.x * NB + b) * d + (size_t)v * VEC);
#pragma unroll
                for (int e4 = 0; e4 < VEC / 4; ++e4)
                    out[e4] = make_float4(acc[b][4 * e4], acc[b][4 * e4 + 1], acc[b][4 * e4 + 2], acc[b][4 * e4 + 3]);
            }
        }
    };
    auto work_rows = [&](auto stream) {
        if constexpr (NB <= 2) {
            if (nvec % (UA / 2 * 64) == 0) return work(stream, std::false_type{});
        }
        work(stream, std::true_type{});
    };
    if (streams(NB, n, d, (int)sizeof(W))) work_rows(std::true_type{});
    else work_rows(std::false_type{});
    store_list();
}

// ---------------------------------------------------------------------------
// y[b][:] = sum over the blocks of the row kernel that had rows (second stage of
// the deterministic down-projection reduction, App. C).
// A block owns RED_COLS float4 columns (one 128-byte line) of one token; the list
// of partials is cut into RED_SEGS contiguous segments summed by different
// threads (at most four partials each, requested together); the eight segments of a wave are then
// combined with lane shifts, the eight waves through LDS.  The order depends
// only on the number of partials: used[1] where a list was used (the row kernels leave its length and that there), else `parts`.
// Bound: two dependent trips, the number and the partials.
// ---------------------------------------------------------------------------
__device__ __forceinline__ float seg8_sum(float v)
{
    v += dpp_move<0x128>(v);        // row_ror:8  -> lanes l and l^8
    return add_xor32(add_xor16(v));
}

__global__ __launch_bounds__(RED_COLS *RED_SEGS) void k_reduce_y(const float *__restrict__ ypart,
                                                                 const int32_t *__restrict__ used, float *__restrict__ y,
                                                                 int parts, int NB, int d)
{
    static_assert(RED_COLS == 8, "a wave holds 8 columns x 8 segments");
    constexpr int PER = ROWS_BLOCKS / RED_SEGS;                    // most partials of a segment
    __shared__ float4 wred[RED_COLS * RED_SEGS / 64][RED_COLS];
    const int gact = used != nullptr ? used[1] : parts;
    const int vpt = d / 4, b = blockIdx.y;
    const int c = threadIdx.x % RED_COLS, seg = threadIdx.x / RED_COLS;
    const int v = blockIdx.x * RED_COLS + c;
    const int per = (gact + RED_SEGS - 1) / RED_SEGS;
    const int g0 = seg * per, g1 = v < vpt ? min(gact, g0 + per) : 0;
    const __amdgpu_buffer_rsrc_t all = range_of(ypart, (uint32_t)(ROWS_BLOCKS * NB) * vpt * 16);
    uint4 p[PER];
#pragma unroll
    for (int q = 0; q < PER; ++q)
        p[q] = load_range(all, g0 + q < g1 ? (uint32_t)(((g0 + q) * NB + b) * vpt + v) * 16u : OUTSIDE);
    float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        const float4 f = as_float4(p[q]);
        s.x += f.x; s.y += f.y; s.z += f.z; s.w += f.w;
    }
    s.x = seg8_sum(s.x); s.y = seg8_sum(s.y); s.z = seg8_sum(s.z); s.w = seg8_sum(s.w);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (lane < RED_COLS) wred[wave][lane] = s;
    __syncthreads();
    if (threadIdx.x < RED_COLS && v < vpt) {
        float4 t = wred[0][c];
#pragma unroll
        for (int q = 1; q < RED_COLS * RED_SEGS / 64; ++q) {
            const float4 w = wred[q][c];
            t.x += w.x; t.y += w.y; t.z += w.z; t.w += w.w;
        }
        reinterpret_cast<float4 *>(y)[(size_t)b * vpt + v] = t;
    }
}

// ---------------------------------------------------------------------------
// Glue of the stacked benchmark: x_next = (x+y)/sqrt(mean((x+y)^2)+eps) + shift.
// One block; the sum of squares is reduced in a fixed order.
// ---------------------------------------------------------------------------
template <typename W>
__global__ __launch_bounds__(256) void k_stack_glue(const W *x, const float *__restrict__ y,
                                                    const float *__restrict__ shift, int d, float eps, W *x_next)
{
    constexpr int VEC = Elem<W>::VEC;
    constexpr int KEEP = 4;                            // vectors of x + y a thread keeps in registers
    __shared__ float part[4];
    const int tid = threadIdx.x, nvec = d / VEC;
    // one trip to memory for x, y and the shift of the thread's first KEEP vectors; the sum of squares in the order that
    // glue_block_total states
    float v[KEEP][VEC], sh[KEEP][VEC];
#pragma unroll
    for (int k = 0; k < KEEP; ++k) {
        const int vi = tid + k * 256;
        if (vi < nvec) {
            load_vec(x + (size_t)vi * VEC, v[k]);
#pragma unroll
            for (int e4 = 0; e4 < VEC / 4; ++e4) {
                const float4 yv = *reinterpret_cast<const float4 *>(y + (size_t)vi * VEC + 4 * e4);
                const float4 sv = *reinterpret_cast<const float4 *>(shift + (size_t)vi * VEC + 4 * e4);
                v[k][4 * e4] += yv.x; v[k][4 * e4 + 1] += yv.y; v[k][4 * e4 + 2] += yv.z; v[k][4 * e4 + 3] += yv.w;
                sh[k][4 * e4] = sv.x; sh[k][4 * e4 + 1] = sv.y; sh[k][4 * e4 + 2] = sv.z; sh[k][4 * e4 + 3] = sv.w;
            }
        }
    }
    float ss = 0.f;
#pragma unroll
    for (int k = 0; k < KEEP; ++k)
        if (tid + k * 256 < nvec) {
#pragma unroll
            for (int e = 0; e < VEC; ++e) ss = fmaf(v[k][e], v[k][e], ss);
        }
    for (int vi = tid + KEEP * 256; vi < nvec; vi += 256) {
        float xv[VEC];
        load_vec(x + (size_t)vi * VEC, xv);
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
            const float a = xv[e] + y[(size_t)vi * VEC + e];
            ss = fmaf(a, a, ss);
        }
    }
    const float tot = glue_block_total(ss, part);      // its barriers: every read of x above is done (x_next may alias x)
    const float inv = 1.0f / sqrtf(tot / (float)d + eps);
    auto emit = [&](int vi, const float (&vv)[VEC], const float (&ss4)[VEC]) {
        W outv[VEC];
#pragma unroll
        for (int e = 0; e < VEC; ++e) from_f32(vv[e] * inv + ss4[e], &outv[e]);
        *reinterpret_cast<uint4 *>(x_next + (size_t)vi * VEC) = *reinterpret_cast<const uint4 *>(outv);
    };
#pragma unroll
    for (int k = 0; k < KEEP; ++k)
        if (tid + k * 256 < nvec) emit(tid + k * 256, v[k], sh[k]);
    for (int vi = tid + KEEP * 256; vi < nvec; vi += 256) {   // a thread rewrites only the vector it reads here
        float xv[VEC], sv[VEC];
        load_vec(x + (size_t)vi * VEC, xv);
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
            xv[e] += y[(size_t)vi * VEC + e];
            sv[e] = shift[(size_t)vi * VEC + e];
        }
        emit(vi, xv, sv);
    }
}

}  // namespace svdp
