// Kernels on the matrix cores.
//
// The FFN over a list of rows for batches of several tokens in bf16 storage (the regime the paper's
// Sec. 6 names as the limit of the sparse path: the union of the tokens' masks is dense enough that a
// row-at-a-time kernel spends its time in per-token vector arithmetic, and App. C's Alg. 4 treats the
// selected rows as a small dense contraction), in two kernels:
//   k_gate_up_mfma  same contract and list handling as k_rows, but it ends with h = ReLU(g) * u of its
//            chunk of the list written to memory (h [list position][NB], and the checked list).  Tiles of 16
//            list rows x 64 elements of d; four lanes fetch 64 contiguous bytes of one row per load, two
//            loads cover 128 bytes and feed two v_mfma_f32_16x16x32_bf16 per matrix, whose other operand is
//            x in LDS.  The eight waves of the block split d between them; their
//            16x16 partial tiles meet in LDS and are added in wave order.
//   k_down_slices   y[token][col] = sum over the list of h * W_downT[row][col], by blocks that own a
//            128-byte column slice and one of eight parts of the list (see there).
// Products of bf16 values are exact in fp32 and every sum has a fixed order.
// Both are bound by the stream and the trips before it: mask and x, the rows; the list's length, its part of the list, the rows.
// 4096 x 14336, eight tokens, 8077 rows on average, weights from memory, launch included: gate/up 132 MB in 27.6 us (4.8 TB/s), slices
// 66 MB in 18.1 us (3.7 TB/s).  So every phase's requests stand together and outside of branches, one step (one group of rows) is under
// way while another is multiplied.  Step of this shape, three layers in turn, with loads in branches in all its kernels -> now: 69.1 ->
// 62.2 us.
// A row's last, partial step (d no multiple of 64) is a step of its own, with zeros past the end on both sides.
// Requirements checked by the host: NB <= 8.
// Dynamic LDS of k_gate_up_mfma: NB * mf_x_stride * 16 bytes (x) + ROWS_WAVES*max_chunk*2*NB floats (partial tiles) +
// max_chunk ints (list); max_chunk % 16 == 0.
#pragma once

#include "svdp_kernels.h"

namespace svdp {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));

constexpr int MF_ROWS = 16;      // list rows per tile
constexpr int DOWN_RG = 8;       // k_down_slices: parts of the list per column slice (= partial outputs) ...
constexpr int DOWN_MIN_CHUNK = 64;     // ... and fewest rows of a part
// LDS of k_gate_up_mfma behind x: partial tiles and the list.
__host__ __device__ constexpr size_t mf_rest_bytes(int D, int NB)
{
    return (size_t)(ROWS_WAVES * 2 * NB + 1) * rows_max_chunk(D, MF_ROWS, MF_ROWS) * 4;
}
// 16-byte vectors from one token's x to the next in LDS: with four more than there are, the four vectors that eight tokens' lanes read at
// once, and the consecutive ones that a wave writes, lie in different banks.  Without them where the layer leaves no room (four tokens,
// d > 16256, D > 28672).
__host__ __device__ constexpr int mf_x_stride(int d, int D, int NB)
{
    const int vectors = (d + 63) / 64 * 8;
    return NB * (vectors + 4) * 16 + mf_rest_bytes(D, NB) <= LDS_MAX ? vectors + 4 : vectors;
}
__host__ __device__ constexpr size_t mf_lds(int d, int D, int NB) { return (size_t)(NB * mf_x_stride(d, D, NB) * 16) + mf_rest_bytes(D, NB); }

__device__ __forceinline__ f32x4_t mfma_bf16(const uint4 &a, const uint4 &b, f32x4_t c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, a), __builtin_bit_cast(bf16x8_t, b), c,
                                                   0, 0, 0);
}

template <int NB, int MODE>
__global__ __launch_bounds__(ROWS_THREADS) void k_gate_up_mfma(
    const bf16 *__restrict__ x, const void *__restrict__ list, const bf16 *__restrict__ Wg, const bf16 *__restrict__ Wu,
    const int32_t *__restrict__ nnz_in, int dB, int D, uint32_t flags, int32_t *__restrict__ idx_out,
    int32_t *__restrict__ nnz_out, int32_t *__restrict__ n_used, float *__restrict__ hbuf, int32_t *__restrict__ lst)
{
    const int d = dB & 0xffff, B = dB >> 16;
    const int max_chunk = rows_max_chunk(D, MF_ROWS, MF_ROWS);
    constexpr int min_chunk = MF_ROWS;
    static_assert(NB == 1 || NB == 2 || NB == 4 || NB == 8, "token slots are addressed with a mask");
    extern __shared__ uint4 smem16[];
    const int full = d / 64, nsteps = (d + 63) / 64;               // 64-element steps per row: whole ones, all
    const int stride = mf_x_stride(d, D, NB);
    uint4 *xs = smem16;                                            // [NB][stride]
    float *part = reinterpret_cast<float *>(xs + NB * stride);     // [ROWS_WAVES][tiles][2][16][NB]
    int *lidx = reinterpret_cast<int *>(part + (size_t)ROWS_WAVES * max_chunk * 2 * NB);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lm = lane & 15, lq = lane >> 4;
    constexpr int G = ROWS_BLOCKS;

    // ---- request the mask words, then x ----
    int lane_first, wpl;
    uint64_t held[ROWS_WREG];
    rows_request_mask<MODE>(D, list, lane, wpl, held);
    uint4 xv[1][NB];
    rows_request_x<bf16, NB>(x, B, d, 0, xv);
    const int n = rows_list_length<MODE>(D, list, nnz_in, lane, wpl, held, lane_first);
    const int chunk = chunk_of(n, G, min_chunk);
    const int lo = min(n, (int)blockIdx.x * chunk);
    const int hi = min(n, lo + chunk);
    const int cnt = hi - lo;
    // written at the kernel's end: a wait for loads waits for the stores in front of them too
    auto store_list = [&] {
        if (blockIdx.x == 0 && tid == 0) {
            if (MODE != ROWS_DENSE)
                *reinterpret_cast<int2 *>(n_used) = make_int2(n, active_blocks(n, chunk_of(n, DOWN_RG, DOWN_MIN_CHUNK)));
            if (MODE == ROWS_MASK && nnz_out != nullptr) *nnz_out = n;
        }
        if (MODE != ROWS_DENSE)
            for (int q = tid; q < cnt; q += ROWS_THREADS) {
                lst[lo + q] = lidx[q];
                if (MODE == ROWS_MASK && idx_out != nullptr) idx_out[lo + q] = lidx[q];
            }
    };
    if (cnt <= 0) {
        store_list();
        return;
    }
    for (int v0 = 0; v0 < nsteps * 8; v0 += ROWS_THREADS) {        // zeros past the row's end
        if (v0 != 0) rows_request_x<bf16, NB>(x, B, d, v0, xv);
#pragma unroll
        for (int b = 0; b < NB; ++b)
            if (v0 + tid < nsteps * 8) xs[b * stride + v0 + tid] = xv[0][b];
    }
    rows_block_list<MODE>(D, list, lane_first, wpl, held, lo, hi, lidx);

    const bool drelu = (flags & 1u) != 0;
    // rows past the end of the chunk repeat its last row, and a rejected entry of the caller's list
    // (-1) reads row 0 in its place; the h of both is zero
    auto row_of = [&](int q) -> size_t {
        const int qq = min(q, cnt - 1);
        return MODE == ROWS_DENSE ? (size_t)(lo + qq) : (size_t)max(lidx[qq], 0);
    };
    const int ntile = (cnt + MF_ROWS - 1) / MF_ROWS;

    // ---- this wave's share of d is the steps [first, last); one is under way while another is multiplied ----
    // (Groups of several steps have to take the last group's place for steps that the wave does not have: weights of zero do not
    // do that, since zero times an infinite x is NaN, and requests for them are not free.  Groups of four -> single steps, eight tokens,
    // a list, weights from memory / the same layer again and again, us: d = 512, n = 2000 15.0 -> 12.9 / 13.4 -> 10.8 (d = 520), d = 1024, n = 1843
    // 15.7 -> 13.2 / 14.3 -> 11.8, d = 2560, n = 1920 20.8 -> 17.4 / 19.9 -> 16.6, d = 4096, n = 3072 23.9 -> 23.3 / 23.5 -> 22.9, d = 6144, n =
    // 4608 46.4 -> 46.9 / 41.5 -> 42.7, n = 11059 90.6 -> 90.0 / 89.5 -> 88.5, d = 8192 level.)
    const int first = wave * nsteps / ROWS_WAVES, end = (wave + 1) * nsteps / ROWS_WAVES, last = min(end, full);
    const int tb = lm & (NB - 1);                                   // token slot read as the x operand
    const uint4 *xt = xs + tb * stride + lq;
    f32x4_t ag = {0.f, 0.f, 0.f, 0.f}, au = {0.f, 0.f, 0.f, 0.f};
    // the tile's last products, and its partial sums: the lane holds rows 4*lq .. 4*lq+3 of the tile for token lm
    auto finish_tile = [&](int t) {
        if (end > full) {                        // the last wave: the partial step
            const size_t row = row_of(t * MF_ROWS + lm);
            const bf16 *pg = Wg + row * d + (size_t)full * 64 + lq * 8, *pu = Wu + row * d + (size_t)full * 64 + lq * 8;
            const uint4 zero = make_uint4(0u, 0u, 0u, 0u);
            const int col = full * 64 + lq * 8;
            const uint4 g0 = col < d ? load_raw(pg) : zero, u0 = col < d ? load_raw(pu) : zero;
            const uint4 g1 = col + 32 < d ? load_raw(pg + 32) : zero, u1 = col + 32 < d ? load_raw(pu + 32) : zero;
            const uint4 xa = xt[full * 8], xb = xt[full * 8 + 4];
            ag = mfma_bf16(g0, xa, ag);
            au = mfma_bf16(u0, xa, au);
            ag = mfma_bf16(g1, xb, ag);
            au = mfma_bf16(u1, xb, au);
        }
        if (lm < NB) {
            float *pt = part + ((size_t)(wave * ntile + t) * 2) * MF_ROWS * NB;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                pt[(lq * 4 + i) * NB + lm] = ag[i];
                pt[MF_ROWS * NB + (lq * 4 + i) * NB + lm] = au[i];
            }
        }
        ag = au = f32x4_t{0.f, 0.f, 0.f, 0.f};
    };
    struct Step {
        uint4 g0, g1, u0, u1;
    };
    if (first >= last) {
        for (int t = 0; t < ntile; ++t) finish_tile(t);
    } else {
        // step s of tile t; past the last tile the matrices' first line: nothing is asked for in a branch, after which every load
        // would have to be awaited at once
        auto request = [&](int t, int s, Step &w) {
            const bool beyond = t >= ntile;
            const size_t row = beyond ? 0 : row_of(t * MF_ROWS + lm), at = row * d + (beyond ? 0 : (size_t)s * 64) + lq * 8;
            w.g0 = load_raw(Wg + at);
            w.g1 = load_raw(Wg + at + 32);
            w.u0 = load_raw(Wu + at);
            w.u1 = load_raw(Wu + at + 32);
            __builtin_amdgcn_sched_barrier(0);
        };
        Step wa, wb;
        int t = 0, s = first, tn = 0, sn = first;                    // the step multiplied, the step requested
        auto advance = [&](int &tt, int &ss) {
            if (++ss >= last) {
                ss = first;
                ++tt;
            }
        };
        auto turn = [&](const Step &now, Step &next) {
            advance(tn, sn);
            request(tn, sn, next);
            const uint4 xa = xt[s * 8], xb = xt[s * 8 + 4];
            ag = mfma_bf16(now.g0, xa, ag);
            au = mfma_bf16(now.u0, xa, au);
            ag = mfma_bf16(now.g1, xb, ag);
            au = mfma_bf16(now.u1, xb, au);
            if (s + 1 >= last) finish_tile(t);
            advance(t, s);
        };
        request(tn, sn, wa);
        while (true) {
            turn(wa, wb);
            if (t >= ntile) break;
            turn(wb, wa);
            if (t >= ntile) break;
        }
    }
    __syncthreads();
    // partial tiles of the waves, added in wave order -> h[list position][token]
    for (int e = tid; e < cnt * NB; e += ROWS_THREADS) {
        const int q = e / NB, b = e % NB;
        float h = 0.f;
        if (MODE != ROWS_LIST || lidx[q] >= 0) {
            const int t = q / MF_ROWS, rr = q % MF_ROWS;
            float gs = 0.f, us = 0.f;
#pragma unroll
            for (int w = 0; w < ROWS_WAVES; ++w) {
                const float *pt = part + ((size_t)(w * ntile + t) * 2) * MF_ROWS * NB;
                gs += pt[rr * NB + b];
                us += pt[MF_ROWS * NB + rr * NB + b];
            }
            h = fmaxf(gs, 0.f) * (drelu ? fmaxf(us, 0.f) : us);
        }
        hbuf[(size_t)(lo + q) * NB + b] = h;
    }
    store_list();
}

// ---------------------------------------------------------------------------
// Down projection over column slices, for batches (Alg. 4's last product; App. C: W_down is stored by columns,
// W_downT [D][d], so that a selected neuron is one contiguous row):
//     y[token][col] = sum over the list of h[position][token] * W_downT[row(position)][col].
// Block (slice, rg) owns the 64 columns (one 128-byte line of every row) [64 slice, +64) and the rg-th of RG equal
// parts of the list, and writes its sums to ypart [rg][NB][d]; k_reduce_y adds the RG parts.  Against one partial
// y per row-kernel block (256 of them: 32 MB written and read again at eight tokens) this leaves RG * NB * d
// floats.  Eight lanes fetch the 128 bytes of a row, so a wave's load instruction covers eight rows; a lane keeps
// NB x 8 sums (its eight columns for every token), and h (written by the gate/up kernel, a few hundred KB that stay
// in L2) is read by position.  The sums over a wave's eight row lanes and then over the waves are taken in a fixed
// order through LDS.
// The last slice may have fewer columns.  Requirement checked by the host: ceil(D / RG) <= DS_MAX_CHUNK.
// ---------------------------------------------------------------------------
constexpr int DS_THREADS = 256;
constexpr int DS_WAVES = DS_THREADS / 64;
constexpr int DS_UB = 4;             // wave loads (eight rows each) in flight, twice while the next group is fetched
constexpr int DS_MAX_CHUNK = 4096;   // list entries of a block kept in LDS
constexpr int DS_LPR = 8;            // lanes per row: 16 bytes each, one 128-byte line
constexpr int DS_SW = DS_LPR * 8;    // columns of a slice

template <int NB, bool DENSE>
__global__ __launch_bounds__(DS_THREADS) __attribute__((amdgpu_waves_per_eu(2))) void k_down_slices(const bf16 *__restrict__ WdT,
                                                            const int32_t *__restrict__ lst,
                                                            const int32_t *__restrict__ n_ptr, int D, int d,
                                                            const float *__restrict__ hbuf, float *__restrict__ ypart)
{
    constexpr int LPR = DS_LPR, SW = DS_SW;
    constexpr int RPW = 64 / LPR;                // rows per wave load
    constexpr int RSETS = RPW / 2;               // row-lane sets of a wave left after the lane shift below
    __shared__ int4 list4[DENSE ? 1 : DS_MAX_CHUNK / 4 + 1];
    __shared__ float red[DS_WAVES * RSETS * NB * SW];         // [DS_WAVES * RSETS][NB][SW]
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int cg = lane % LPR, sub = lane / LPR;
    const int slice = blockIdx.x, rg = blockIdx.y;
    int n = n_ptr != nullptr ? *n_ptr : D;
    n = max(0, min(n, D));
    const int chunk = chunk_of(n, DOWN_RG, DOWN_MIN_CHUNK);
    const int lo = min(n, rg * chunk), hi = min(n, lo + chunk), cnt = hi - lo;
    if (cnt <= 0) return;
    // the part of the list, in whole 16-byte vectors (D is a multiple of four): at most five a thread, one trip for all
    const int lo4 = lo / 4, off = lo % 4;
    if (!DENSE) {
        constexpr int LV = DS_MAX_CHUNK / 4 / DS_THREADS;
        const __amdgpu_buffer_rsrc_t entries = range_of(lst, (uint32_t)D * 4);
        const int n4 = (hi + 3) / 4 - lo4;
        uint4 e[LV + 1];
#pragma unroll
        for (int k = 0; k <= LV; ++k) {
            const int v = tid + k * DS_THREADS;
            e[k] = load_range(entries, v < n4 ? (uint32_t)(lo4 + v) * 16u : OUTSIDE);
        }
#pragma unroll
        for (int k = 0; k <= LV; ++k) {
            const int v = tid + k * DS_THREADS;
            if (v < n4) list4[v] = __builtin_bit_cast(int4, e[k]);
        }
        __syncthreads();
    }
    const int *lidx = reinterpret_cast<const int *>(list4) + off;
    const int ngroups = (cnt + RPW - 1) / RPW;
    const bool colok = slice * SW + cg * 8 < d;
    const bf16 *colp = WdT + (size_t)slice * SW + (size_t)(colok ? cg : 0) * 8;

    // v_mfma_f32_4x4x1_16b: sixteen independent 4 x 4 outer products; the four lanes of a block work on the same
    // row, lane j of the block supplies h of token 4 tg + j and its own column's weight, and keeps the four tokens'
    // sums for its own column: acc[tg][e][i] belongs to token 4 tg + i and column 8 cg + e.
    constexpr int TG = (NB + 3) / 4;
    f32x4_t acc[TG][8];
#pragma unroll
    for (int g = 0; g < TG; ++g)
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[g][e] = f32x4_t{0.f, 0.f, 0.f, 0.f};

    // group g of the chunk = its rows RPW g .. RPW g + RPW - 1; this wave takes the groups wave, wave + DS_WAVES, ...
    // Requested without branches (each load inside of one is waited for): positions past the end and rejected entries of the
    // caller's list read another row, whose weights are then replaced by zeros (h is zero already, but a weight may be infinite).
    const __amdgpu_buffer_rsrc_t hpart = range_of(hbuf, (uint32_t)hi * NB * 4);
    const uint32_t my_token = (lane & 3) < NB ? (uint32_t)(lane & 3) * 4u : OUTSIDE;
    struct Group {
        uint4 w[DS_UB];
        float h[DS_UB][TG];
        bool in[DS_UB];
    };
    auto work = [&](auto stream) {
        constexpr bool STREAM = decltype(stream)::value;
        auto fetch = [&](int g0, Group &p) {
            int row[DS_UB];
#pragma unroll
            for (int k = 0; k < DS_UB; ++k) {
                const int q = (g0 + k * DS_WAVES) * RPW + sub;
                row[k] = DENSE ? lo + min(q, cnt - 1) : lidx[min(q, cnt - 1)];
                p.in[k] = colok && q < cnt && row[k] >= 0;
            }
#pragma unroll
            for (int k = 0; k < DS_UB; ++k) {
                const int q = (g0 + k * DS_WAVES) * RPW + sub;
                p.w[k] = load_raw_hint<STREAM>(colp + (size_t)max(row[k], 0) * d);
                const uint32_t at = NB < 4 && my_token == OUTSIDE ? OUTSIDE : (uint32_t)((lo + q) * NB) * 4u + my_token;
#pragma unroll
                for (int g = 0; g < TG; ++g)
                    p.h[k][g] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(hpart, at, g * 16, 0));
            }
            __builtin_amdgcn_sched_barrier(0);
        };
        auto consume = [&](const Group &p) {
#pragma unroll
            for (int k = 0; k < DS_UB; ++k) {
                float w[8];
                const uint4 in = make_uint4(p.in[k] ? p.w[k].x : 0u, p.in[k] ? p.w[k].y : 0u, p.in[k] ? p.w[k].z : 0u, p.in[k] ? p.w[k].w : 0u);
                widen(in, w, (const bf16 *)nullptr);
#pragma unroll
                for (int e = 0; e < 8; ++e)
#pragma unroll
                    for (int g = 0; g < TG; ++g)
                        acc[g][e] = __builtin_amdgcn_mfma_f32_4x4x1f32(p.h[k][g], w[e], acc[g][e], 0, 0, 0);
            }
        };
        Group pa, pb;
        constexpr int STEP = DS_WAVES * DS_UB;
        if (wave < ngroups) fetch(wave, pa);
        for (int g0 = wave; g0 < ngroups; g0 += 2 * STEP) {
            fetch(g0 + STEP, pb);                // past the end: the last row again, not counted
            consume(pa);
            if (g0 + STEP >= ngroups) break;
            fetch(g0 + 2 * STEP, pa);
            consume(pb);
        }
    };
    if (streams(8, n, d, 2)) work(std::true_type{});            // whatever NB: on the engine's own choice it is 8
    else work(std::false_type{});
    // row lanes l and l ^ 8 first (a lane shift), then the four remaining sets of a wave and the waves through
    // LDS, in order
#pragma unroll
    for (int g = 0; g < TG; ++g)
#pragma unroll
        for (int e = 0; e < 8; ++e)
#pragma unroll
            for (int i = 0; i < 4; ++i) acc[g][e][i] += dpp_move<0x128>(acc[g][e][i]);           // row_ror:8
    if ((sub & 1) == 0) {
        const int set = wave * RSETS + (sub >> 1);
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int e = 0; e < 8; ++e) red[(set * NB + b) * SW + cg * 8 + e] = acc[b / 4][e][b % 4];
    }
    __syncthreads();
    for (int o = tid; o < NB * SW; o += DS_THREADS) {
        const int b = o / SW, c = o % SW;
        if (slice * SW + c >= d) continue;
        float t = 0.f;
#pragma unroll
        for (int p = 0; p < DS_WAVES * RSETS; ++p) t += red[(p * NB + b) * SW + c];
        ypart[((size_t)rg * NB + b) * d + (size_t)slice * SW + c] = t;
    }
}

// ---------------------------------------------------------------------------
// Predictor stage 2 on the matrix cores: s_i = t . Q[i,:] + b_i for a slab of
// 64 neurons and up to eight tokens, and the slab's mask word (eq. 2).  One
// wave per 16 rows of Q; a lane fetches 16 bytes of one row per column block (four lanes: 64
// contiguous bytes; KB blocks are requested behind the partials of t).  t is the sum of the nt
// stage-1 partials and lies in LDS in operand order:
//   fp32: as it is, v_mfma_f32_16x16x4_f32;
//   bf16: split into three bf16 terms hi + mid + lo = t exactly to 24 bits, so that bf16
//         MFMAs give fp32-accurate scores: every product is exact and the accumulation is fp32.  An infinite t or NaN is hi,
//         with mid = lo = 0.  An infinite Q times a zero mid or lo is NaN, and the terms' products may overflow where t's
//         does not: a score that is not finite is worked out again from t = (mid + lo) + hi by fp32 arithmetic.
// Columns past r are zeros on both sides, so every rank that a layer may have is taken.
//
// Bound: the chain launch, partials of t, operands, MFMAs; the bytes of Q are half of it at most.  Taken for fp32 and for
// ranks that are no multiple of 32 as well: a row's sum over its columns is one accumulator here, where the vector kernel needs
// six lane exchanges per row and token (and k_tsum before it: 2 to 4.6 us).  Step with three and more tokens, vector kernel
// -> this one, in us: fp32 d = 464, D = 2176, r = 192, three tokens 22.7 -> 17.7 (scores 10.2 -> 5.1); fp32 d = 1720, D = 8064,
// r = 464, six tokens 52.4 -> 41.0 (20.7 -> 11.2); bf16 d = 512, D = 2240, r = 24, four tokens 22.0 -> 17.9.
// Partials of t are requested NT at a time and in front of Q, as ranges: in groups of four behind Q each group's wait was for Q as well.
// A request past the last partial or the row's end is not free, so NT (4, 8, 16) and KB (4, 8, 12, 16) follow what there is.  t = x P and scores,
// NT = 16 and KB = 4, 8, 16 -> this, us: 256 x 1024, r = 32, four tokens 5.8 -> 5.0, 1024 x 4096, r = 256, eight tokens 7.8 -> 6.9, 2048 x 8192, r =
// 384, eight tokens 10.2 -> 9.1, 5120 x 13824, r = 320, eight tokens (20 partials, three times eight instead of twice sixteen) 12.4 -> 11.3.
// Step of 4096 x 14336, r = 256, eight tokens 63.1 -> 62.0 / 60.5 -> 59.7 us (two boxes), of 3584 x 18944, r = 512, four tokens level.
// Tried on it: two waves per 16 rows with half of the columns each, the blocks of two slabs in one (the same), column blocks in another
// order per wave (0.4 slower),
// the compiler's own unrolling of the partials' loop (eight tokens, r = 256: 6.7 -> 9.2).
// Dynamic LDS: scm_lds bytes.
// ---------------------------------------------------------------------------
constexpr int SCM_THREADS = 256;
constexpr int SCM_KB = 16;          // most column blocks of Q held in registers
constexpr int SCM_NT = 16;          // most partials of t requested together

// a and b as hi + mid + lo each, two bf16 to a word.  Rounded by the packed conversion instead of
// in integer arithmetic (step of bf16 d = 512, D = 2240, r = 24, four tokens 17.3 -> 16.6 us, d = 1024, D = 4096, r = 256, three
// tokens 18.0 -> 17.5).  WIDE: also where an element is infinite or NaN (then hi, with
// mid = lo = 0) or rounds past the largest bf16 (then hi is that).
constexpr float BF16_MAX = 0x1.fep127f;
template <bool WIDE>
__device__ __forceinline__ void split3(float a, float b, uint32_t &hi, uint32_t &mid, uint32_t &lo)
{
    typedef float f32x2_t __attribute__((ext_vector_type(2)));
    auto pack = [](float x, float y) { return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2_t{x, y}), bf16x2_t)); };
    auto capped = [](float v) { return WIDE && __builtin_isfinite(v) ? fminf(fmaxf(v, -BF16_MAX), BF16_MAX) : v; };
    hi = pack(capped(a), capped(b));
    float ra = a - __uint_as_float(hi << 16), rb = b - __uint_as_float(hi & 0xffff0000u);
    if (WIDE) {
        ra = __builtin_isfinite(a) ? ra : 0.f;
        rb = __builtin_isfinite(b) ? rb : 0.f;
    }
    mid = pack(ra, rb);
    lo = pack(ra - __uint_as_float(mid << 16), rb - __uint_as_float(mid & 0xffff0000u));
}

__device__ __forceinline__ f32x4_t mfma_f32(const uint4 &a, const uint4 &b, f32x4_t c)
{
    c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.x), __uint_as_float(b.x), c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.y), __uint_as_float(b.y), c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.z), __uint_as_float(b.z), c, 0, 0, 0);
    return __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.w), __uint_as_float(b.w), c, 0, 0, 0);
}

template <typename W>
constexpr int scm_block() { return 4 * Elem<W>::VEC; }                    // columns of a block
template <typename W>
constexpr int scm_terms() { return Elem<W>::BYTES == 2 ? 3 : 1; }         // 16-byte operands per column group and token
template <typename W>
size_t scm_lds(int NB, int r)
{
    const size_t nkb = (r + scm_block<W>() - 1) / scm_block<W>();
    return scm_terms<W>() * nkb * 4 * NB * 16;
}

template <typename W, int NB, int KB, int NT>
__global__ __launch_bounds__(SCM_THREADS) __attribute__((amdgpu_waves_per_eu(2))) void k_scores_mfma(
    const W *__restrict__ Q, const float *__restrict__ bias, const float *__restrict__ tpart, int nt, int r, int B,
    uint64_t *__restrict__ mask_out, float *__restrict__ s_out, int D)
{
    static_assert(NB == 1 || NB == 2 || NB == 4 || NB == 8, "token slots are addressed with a mask");
    constexpr int VEC = Elem<W>::VEC, CB = scm_block<W>(), TERMS = scm_terms<W>();
    extern __shared__ uint4 smem16[];
    __shared__ uint32_t word16[SCM_THREADS / 64];
    uint4 *ops = smem16;                                            // [TERMS][nkb * 4 column groups][NB]
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lm = lane & 15, lq = lane >> 4;
    const int i0 = blockIdx.x * SC_SLAB + wave * 16;
    const int nkb = (r + CB - 1) / CB;

    // partials p0 .. p0 + NT - 1 of t for slot u = (token b, columns VEC g .. VEC g + VEC - 1); zeros past the last
    const int ngr = r / VEC, slots = nkb * 4, all = NB * slots;
    const __amdgpu_buffer_rsrc_t parts = range_of(tpart, (uint32_t)(nt * NB * r) * 4);
    uint4 v[NT][VEC / 4];
    auto request_t = [&](int u, int p0) {
        const int b = u / slots, g = u - b * slots;
        const uint32_t at = u < all && g < ngr ? (uint32_t)((p0 * NB + b) * r + g * VEC) * 4u : 1u << 31;      // past the range with all k
#pragma unroll
        for (int k = 0; k < NT; ++k)
#pragma unroll
            for (int h = 0; h < VEC / 4; ++h)
                v[k][h] = load_range(parts, at + (uint32_t)(k * NB * r + 4 * h) * 4u);
    };
    request_t(tid, 0);

    uint4 q[KB];
    const __amdgpu_buffer_rsrc_t qrows = range_of(Q + (size_t)i0 * r, (uint32_t)(16 * r) * sizeof(W));
    auto request_q = [&](int kb0) {
#pragma unroll
        for (int k = 0; k < KB; ++k) {
            const int col = (kb0 + k) * CB + lq * VEC;
            q[k] = load_range(qrows, col < r ? (uint32_t)(lm * r + col) * sizeof(W) : OUTSIDE);
        }
    };
    request_q(0);
    float bs[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) bs[i] = bias[i0 + lq * 4 + i];
    __builtin_amdgcn_sched_barrier(0);

    // t of a slot: sum of its partials in order, then its operands
    auto finish_t = [&](int u) {
        const int b = u / slots, g = u - b * slots;
        float t[VEC];
#pragma unroll
        for (int e = 0; e < VEC; ++e) t[e] = 0.f;
        auto add = [&] {
#pragma unroll
            for (int k = 0; k < NT; ++k)
#pragma unroll
                for (int h = 0; h < VEC / 4; ++h) {
                    const float4 p = as_float4(v[k][h]);
                    t[4 * h] += p.x; t[4 * h + 1] += p.y; t[4 * h + 2] += p.z; t[4 * h + 3] += p.w;
                }
        };
        add();                                   // apart from the loop: waits for its own loads only, not for Q
        for (int p0 = NT; p0 < nt; p0 += NT) {
            request_t(u, p0);
            add();
        }
        if (u >= all) return;
        uint4 *op = ops + (size_t)g * NB + b;
        if constexpr (TERMS == 1) {
            *op = make_uint4(__float_as_uint(t[0]), __float_as_uint(t[1]), __float_as_uint(t[2]), __float_as_uint(t[3]));
        } else {
            float top = 0.f;
#pragma unroll
            for (int e = 0; e < VEC; ++e) top = fmaxf(top, fabsf(t[e]));
            uint32_t pl[3][VEC / 2];
            if (__builtin_expect(!(top <= BF16_MAX), 0)) {
#pragma unroll
                for (int e = 0; e < VEC / 2; ++e) split3<true>(t[2 * e], t[2 * e + 1], pl[0][e], pl[1][e], pl[2][e]);
            } else {
#pragma unroll
                for (int e = 0; e < VEC / 2; ++e) split3<false>(t[2 * e], t[2 * e + 1], pl[0][e], pl[1][e], pl[2][e]);
            }
#pragma unroll
            for (int p = 0; p < 3; ++p) op[(size_t)p * slots * NB] = make_uint4(pl[p][0], pl[p][1], pl[p][2], pl[p][3]);
        }
    };
    finish_t(tid);
    for (int u = tid + SCM_THREADS; u - tid < all; u += SCM_THREADS) {
        request_t(u, 0);
        finish_t(u);
    }
    __syncthreads();

    f32x4_t acc = {0.f, 0.f, 0.f, 0.f};
    const uint4 *op0 = ops + (size_t)lq * NB + (lm & (NB - 1));
    for (int kb0 = 0; kb0 < nkb; kb0 += KB) {
        if (kb0 > 0) request_q(kb0);
#pragma unroll
        for (int k = 0; k < KB; ++k) {
            if (kb0 + k < nkb) {
                const uint4 *op = op0 + (size_t)(kb0 + k) * 4 * NB;
                if constexpr (TERMS == 1) {
                    acc = mfma_f32(q[k], *op, acc);
                } else {
#pragma unroll
                    for (int p = 0; p < 3; ++p) acc = mfma_bf16(q[k], op[(size_t)p * slots * NB], acc);
                }
            }
        }
    }
    if constexpr (TERMS == 3) {
        const bool plain = __builtin_isfinite(acc[0]) && __builtin_isfinite(acc[1]) && __builtin_isfinite(acc[2]) &&
                           __builtin_isfinite(acc[3]);
        if (__builtin_expect(__any(!plain), 0)) {                   // see above: such scores once more, from t itself
#pragma unroll 1
            for (int i = 0; i < 4; ++i) {
                const W *row = Q + (size_t)(i0 + lq * 4 + i) * r;
                const uint4 *op = ops + (lm & (NB - 1));
                float v = 0.f;
#pragma unroll 1
                for (int g = 0; g < ngr; ++g, op += NB) {
                    float qv[VEC], hi[VEC], mid[VEC], lo[VEC];
                    widen(load_raw(row + (size_t)g * VEC), qv, (const W *)nullptr);
                    widen(op[0], hi, (const W *)nullptr);
                    widen(op[(size_t)slots * NB], mid, (const W *)nullptr);
                    widen(op[(size_t)2 * slots * NB], lo, (const W *)nullptr);
#pragma unroll
                    for (int e = 0; e < VEC; ++e) v = fmaf((mid[e] + lo[e]) + hi[e], qv[e], v);
                }
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    if (k == i && !__builtin_isfinite(acc[k])) acc[k] = v;
            }
        }
    }
    // the lane holds rows i0 + 4*lq .. +3 for token lm
    const float sv[4] = {acc[0] + bs[0], acc[1] + bs[1], acc[2] + bs[2], acc[3] + bs[3]};
    if (s_out != nullptr && lm < B) {
#pragma unroll
        for (int i = 0; i < 4; ++i) s_out[(size_t)lm * D + i0 + lq * 4 + i] = sv[i];
    }
    if (mask_out != nullptr) {
        uint32_t w16 = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint64_t on = __ballot(lm < B && sv[i] > 0.f);
#pragma unroll
            for (int qq = 0; qq < 4; ++qq)
                if ((on >> (16 * qq)) & 0xffffull) w16 |= 1u << (4 * qq + i);
        }
        if (lane == 0) word16[wave] = w16;
        __syncthreads();
        if (tid == 0)
            mask_out[blockIdx.x] = (uint64_t)word16[0] | ((uint64_t)word16[1] << 16) | ((uint64_t)word16[2] << 32) |
                                   ((uint64_t)word16[3] << 48);
    }
}

}   // namespace svdp
