// Statistics of a calibration set for the bias calibration (first two lines of
// Alg. 2): damage weights w[i][t] = |ReLU(W_gate[i,:] x_t) (W_up[i,:] x_t)|^2 ||W_down[:,i]||^2
// and proxy scores s[i][t] = (A B x_t)_i, for T tokens at once.  These are dense
// contractions with reuse (every weight element meets every token), so they run
// on the matrix cores, C = A B^T with both operands stored K-contiguous:
//   k_gemm_nt    t = X P (against P transposed once), 128 x 128 tiles, parts of K; t split into three bf16 terms;
//   k_gemm_wide  gate and up against the tokens (two A operands share the B tiles), epilogue -> w; and, in the same
//                launch, scores = Q against the three terms of t (Q's columns wrap around every r), which is exact to
//                fp32 as in k_scores_mfma.
#pragma once

#include "svdp_rows_mfma.h"

namespace svdp {

constexpr int GM_BM = 128, GM_BN = 128, GM_BK = 64;
constexpr int GM_THREADS = 256;
constexpr int GM_STRIDE = GM_BK / 8 + 1;          // 16-byte chunks per LDS row
constexpr int GM_CPT = GM_BM * (GM_BK / 8) / GM_THREADS;     // chunks per thread and tile (4)

enum GemmEpilogue { EPI_SPLIT3 = 0, EPI_PLAIN = 1 };

__device__ __forceinline__ uint32_t bf16_rne_bits(float v)
{
    bf16 h;
    from_f32(v, &h);
    return h.bits;
}

// c as three bf16 terms, hi + mid + lo = c to 24 bits, at p[0], p[stride], p[2 * stride]
__device__ __forceinline__ void store_split3(float c, uint16_t *__restrict__ p, int stride)
{
    const uint32_t hi = bf16_rne_bits(c);
    const float r1 = c - __uint_as_float(hi << 16);
    const uint32_t mid = bf16_rne_bits(r1);
    const float r2 = r1 - __uint_as_float(mid << 16);
    p[0] = (uint16_t)hi;
    p[stride] = (uint16_t)mid;
    p[2 * stride] = (uint16_t)bf16_rne_bits(r2);
}

// planes[m][3 N] = the sum of the parts [nz][M][N] (in order), split into three bf16 terms
__global__ __launch_bounds__(256) void k_sum_split3(const float *__restrict__ parts, int nz, int M, int N,
                                                    uint16_t *__restrict__ planes)
{
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x, all = (size_t)M * N;
    if (i >= all) return;
    float c = 0.f;
    for (int z = 0; z < nz; ++z) c += parts[(size_t)z * all + i];
    store_split3(c, planes + i / N * (3 * (size_t)N) + i % N, N);
}

// out[i] = sum_j W[i][j]^2 for a bf16 matrix [rows][cols], one wave per row (fixed order): block `block` of
// ceil(rows / NORM_ROWS).
constexpr int NORM_ROWS = GM_THREADS / 64;
struct NormJob {
    const bf16 *W;
    int rows, cols;
    float *out;
};
__device__ __forceinline__ void row_norm2(const NormJob &job, int block)
{
    const int lane = threadIdx.x & 63;
    const int row = block * NORM_ROWS + (threadIdx.x >> 6);
    if (row >= job.rows) return;
    const bf16 *src = job.W + (size_t)row * job.cols;
    const int nvec = job.cols / 8;
    constexpr int AHEAD = 8;                                       // few waves fit beside the product's blocks
    float acc = 0.f;
    for (int v0 = lane; v0 < nvec; v0 += 64 * AHEAD) {
        uint4 raw[AHEAD];
#pragma unroll
        for (int k = 0; k < AHEAD; ++k) raw[k] = v0 + 64 * k < nvec ? load_raw(src + (size_t)(v0 + 64 * k) * 8) : make_uint4(0u, 0u, 0u, 0u);
#pragma unroll
        for (int k = 0; k < AHEAD; ++k) {
            float w[8];
            widen(raw[k], w, (const bf16 *)nullptr);
#pragma unroll
            for (int e = 0; e < 8; ++e) acc = fmaf(w[e], w[e], acc);
        }
    }
    acc = wave_sum(acc);
    if (lane == 0) job.out[row] = acc;
}

// C[m][n] = sum_k A[m][k] * B[n][k], k < K.  A: [M][lda], B: [N][ldb], bf16.
// EPI_SPLIT3: C -> three bf16 terms at planes[m*ldo + {0, N, 2N} + n]
// EPI_PLAIN : out[m*ldo + n] = C; nz parts of K, `kpart` (a multiple of 8) each, part z to out + z*M*ldo
// The blocks behind the product's nx * ny * nz take row norms, which only the launch after this one's needs: the product
// leaves the memory idle and the norms the matrix cores (7B shape, 2048 tokens: 21.6 + 16.8 us as two launches, 28.9 as one; 36 with one load of a row in flight at a time).
template <int EPI>
__global__ __launch_bounds__(GM_THREADS, 2) void k_gemm_nt(const bf16 *__restrict__ A, int lda, const bf16 *__restrict__ Bm,
                                                        int ldb, int M, int N, int K, float *__restrict__ out,
                                                        uint16_t *__restrict__ planes, int ldo, int kpart, int nx, int ny, int nz,
                                                        NormJob norm)
{
    const int block = blockIdx.x;
    if (block >= nx * ny * nz) {
        row_norm2(norm, block - nx * ny * nz);
        return;
    }
    const int bx = block % nx, by = block / nx % ny, bz = block / (nx * ny);
    __shared__ uint4 sA[GM_BM * GM_STRIDE];
    __shared__ uint4 sB[GM_BN * GM_STRIDE];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int lm = lane & 15, lq = lane >> 4;
    const int wm = wave >> 1, wn = wave & 1;
    const int m0 = by * GM_BM, n0 = bx * GM_BN;

    f32x4_t acc[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};

    const int k_begin = bz * kpart, k_end = min(K, k_begin + kpart);
    uint4 ra[GM_CPT], rb[GM_CPT];
    auto fetch = [&](int k0) {
#pragma unroll
        for (int q = 0; q < GM_CPT; ++q) {
            const int id = tid + q * GM_THREADS, row = id >> 3, c = id & 7;
            const int k = k0 + c * 8, m = m0 + row, n = n0 + row;
            const uint4 zero = make_uint4(0u, 0u, 0u, 0u);
            ra[q] = (k < k_end && m < M) ? load_raw(A + (size_t)m * lda + k) : zero;
            rb[q] = (k < k_end && n < N) ? load_raw(Bm + (size_t)n * ldb + k) : zero;
        }
    };
    fetch(k_begin);
    for (int k0 = k_begin; k0 < k_end; k0 += GM_BK) {
        __syncthreads();                                            // the previous step's reads are done
#pragma unroll
        for (int q = 0; q < GM_CPT; ++q) {
            const int id = tid + q * GM_THREADS, row = id >> 3, c = id & 7;
            sA[row * GM_STRIDE + c] = ra[q];
            sB[row * GM_STRIDE + c] = rb[q];
        }
        __syncthreads();
        if (k0 + GM_BK < k_end) fetch(k0 + GM_BK);
#pragma unroll
        for (int h = 0; h < GM_BK / 32; ++h) {
            uint4 fb[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) fb[j] = sB[(wn * 64 + j * 16 + lm) * GM_STRIDE + h * 4 + lq];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const uint4 fa = sA[(wm * 64 + i * 16 + lm) * GM_STRIDE + h * 4 + lq];
#pragma unroll
                for (int j = 0; j < 4; ++j) acc[i][j] = mfma_bf16(fa, fb[j], acc[i][j]);
            }
        }
    }

    if (EPI == EPI_PLAIN) out += (size_t)bz * M * ldo;
    // the lane holds rows 4*lq .. 4*lq+3 and column lm of each 16 x 16 tile
#pragma unroll
    for (int i = 0; i < 4; ++i) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int m = m0 + wm * 64 + i * 16 + lq * 4 + e;
            if (m >= M) continue;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int n = n0 + wn * 64 + j * 16 + lm;
                if (n >= N) continue;
                if (EPI == EPI_PLAIN) out[(size_t)m * ldo + n] = acc[i][j][e];
                else store_split3(acc[i][j][e], planes + (size_t)m * ldo + n, N);
            }
        }
    }
}

// ---------------------------------------------------------------------------
// The large contractions: a block of eight waves takes 256 rows of A (or 128 of each of two A) by 256 of B, one block per
// compute unit.
// Bound: the matrix cores want 64 products per wave and 32-deep K step (1024 cycles for the two waves of a SIMD) while
// the operands are 12 LDS reads per wave (768 cycles of the compute unit's LDS) and 32 KB written into it (256): a
// smaller block is LDS bound, and a block that waits for its own loads between two barriers leaves the cores idle.  So
// four LDS stages of 32 KB are filled straight from memory, three K steps ahead, with ONE barrier per step; the wait in
// front of it only asks for the oldest stage.  (The loads are written by hand because the compiler puts a wait for all of
// them in front of every LDS read.)
// LDS: rows of 64 bytes, the 16-byte chunk c of row i at slot c ^ ((i >> 1) & 3): any eight rows of an operand read fall
// on different banks, and a wave's load still fills 1024 consecutive bytes.
// Blocks are numbered so that a die works on neighbouring tiles (shared rows of A and B stay in its L2).
// Measured (gate and up of d = 4096, D = 11008 against 2048 tokens, 369 GFLOP): 510 us with 128 x 128 tiles, two barriers
// and loads through registers, 398 us so, 379 us with the next step's first operands read ahead (0.97 PFLOP/s; a library
// product of 8192^3 reaches 1.15 here); with the scores (64 us of their own before) in the same launch 443 us for both.
// It is the faster one down to 100 tokens (d = 4096: 149 against 177 us a call, d = 256: 38 against 43 us at 4096 tokens).
// ---------------------------------------------------------------------------
constexpr int GW_THREADS = 512;
constexpr int GW_BK = 32, GW_STAGES = 4;
constexpr int GW_ROWS = 256;                               // of A, and of B
constexpr int GW_STAGE_BYTES = 2 * GW_ROWS * GW_BK * 2;
constexpr int GW_LDS = GW_STAGES * GW_STAGE_BYTES;

typedef __attribute__((address_space(3))) void lds_void_t;

// 64 lanes x 16 bytes from `src` (per lane) to LDS bytes [at, at + 1024); `at` uniform.  Not counted by the compiler:
// the caller waits on vmcnt before a barrier.  m0 is named as written: the compiler does not allocate it, but sets it itself in
// front of the few instructions that read it, and may only do without where it knows who else writes it.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"        // "reserved register"
__device__ __forceinline__ void load_to_lds(const void *src, uint32_t at)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(at), "v"(src) : "m0", "memory");
}
#pragma clang diagnostic pop

// Every wave's LDS reads and all but the newest N of its loads to LDS are done, in all waves of the block.
template <int N>
__device__ __forceinline__ void stage_barrier()
{
    static_assert(N == 0 || N == 4);
    if (N == 4) asm volatile("s_waitcnt vmcnt(4) lgkmcnt(0)\n\ts_barrier" ::: "memory");
    else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// One product of the launch, arguments as in k_gemm_nt.  A2 != nullptr: 128 rows of A1 and of A2 against the same
// columns, out = (max(c1,0)*c2)^2 * scale; else 256 rows of A1, out = c1.
struct WideJob {
    const bf16 *A1, *A2, *B;
    int lda, Ka, ldb, M, N, K;
    const float *scale;
    float *out;
    int ldo, tn, tiles;         // tiles of N, of the whole product
    int direct;                 // K steps that are loaded straight into LDS (none where an operand is not 16-byte aligned)
};
inline WideJob wide_job(const bf16 *A1, const bf16 *A2, int lda, int Ka, const bf16 *B, int ldb, int M, int N, int K,
                        const float *scale, float *out, int ldo)
{
    const int bm = A2 != nullptr ? GW_ROWS / 2 : GW_ROWS, tn = (N + GW_ROWS - 1) / GW_ROWS;
    const bool aligned = ((reinterpret_cast<uintptr_t>(A1) | reinterpret_cast<uintptr_t>(A2) | reinterpret_cast<uintptr_t>(B)) & 15) == 0;
    return WideJob{A1, A2, B, lda, Ka, ldb, M, N, K, scale, out, ldo, tn, (M + bm - 1) / bm * tn, aligned ? K / GW_BK : 0};
}

// Two products in one launch, the tiles of `first` before those of `second`: the short tiles of the scores fill the
// compute units that the last, partly empty round of the long ones leaves idle.
__global__ __launch_bounds__(GW_THREADS, 2) void k_gemm_wide(WideJob first, WideJob second)
{
    extern __shared__ uint4 gw_smem[];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int lm = lane & 15, lq = lane >> 4, wm = wave >> 2, wn = wave & 3;
    const bool is_second = (int)blockIdx.x >= first.tiles;
    const WideJob &job = is_second ? second : first;
    const bf16 *A1 = job.A1, *A2 = job.A2, *Bm = job.B;
    const int lda = job.lda, Ka = job.Ka, ldb = job.ldb, M = job.M, N = job.N, K = job.K;
    // the q-th of a die's consecutive tiles (workgroups go round the dies)
    const int id = (int)blockIdx.x - (is_second ? first.tiles : 0);
    const int die = id & 7, q8 = job.tiles >> 3, rem = job.tiles & 7;
    const int tile = die * q8 + min(die, rem) + (id >> 3);
    const bool pair = A2 != nullptr;
    const int m0 = tile / job.tn * (pair ? GW_ROWS / 2 : GW_ROWS), n0 = tile % job.tn * GW_ROWS;

    // this thread's four chunks of a stage: rows tid / 4 and 128 more of A, the same of B; rows past the end repeat the
    // last one: their results are not stored
    const int row = tid >> 2, chunk = (tid & 3) ^ ((row >> 1) & 3);
    const bf16 *pa0 = A1 + (size_t)min(m0 + row, M - 1) * lda;
    const bf16 *pa1 = pair ? A2 + (size_t)min(m0 + row, M - 1) * lda : A1 + (size_t)min(m0 + 128 + row, M - 1) * lda;
    const bf16 *pb0 = Bm + (size_t)min(n0 + row, N - 1) * ldb;
    const bf16 *pb1 = Bm + (size_t)min(n0 + 128 + row, N - 1) * ldb;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_void_t *)gw_smem;
    const uint32_t piece = __builtin_amdgcn_readfirstlane(lds0 + wave * 1024);
    const int nk = (K + GW_BK - 1) / GW_BK, nfull = job.direct;

    auto a_col = [&](int k) {                               // A's columns repeat every Ka, K <= 3 Ka
        if (k >= Ka) k -= Ka;
        if (k >= Ka) k -= Ka;
        return k;
    };
    auto fill_full = [&](int kt) {
        const int k = kt * GW_BK + chunk * 8, ka = a_col(k);
        const uint32_t at = piece + (kt & (GW_STAGES - 1)) * GW_STAGE_BYTES;
        load_to_lds(pa0 + ka, at);
        load_to_lds(pa1 + ka, at + 8192);
        load_to_lds(pb0 + k, at + 16384);
        load_to_lds(pb1 + k, at + 24576);
    };
    auto fill = [&](int kt) {
        if (kt < nfull) {
            fill_full(kt);
        } else if (kt < nk) {                               // the ragged end of K, zeros beyond it; unaligned operands
            const int k = kt * GW_BK + chunk * 8, ka = a_col(k);
            uint4 v[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = make_uint4(0u, 0u, 0u, 0u);
            if (k < K) {
                v[0] = load_raw(pa0 + ka);
                v[1] = load_raw(pa1 + ka);
                v[2] = load_raw(pb0 + k);
                v[3] = load_raw(pb1 + k);
            }
            uint4 *dst = gw_smem + (kt & (GW_STAGES - 1)) * (GW_STAGE_BYTES / 16) + tid;
#pragma unroll
            for (int e = 0; e < 4; ++e) dst[e * 512] = v[e];
        }
    };

    // a wave's tile t: rows (t / 4) * 128 + wm * 64 + (t % 4) * 16 of the block's 256
    f32x4_t acc[8][4];
#pragma unroll
    for (int t = 0; t < 8; ++t)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[t][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};

    const uint4 *frag = gw_smem + lm * 4 + (lq ^ ((lm >> 1) & 3));        // this lane's place in a 16-row tile
    auto stage = [&](int kt) { return frag + (kt & (GW_STAGES - 1)) * (GW_STAGE_BYTES / 16); };
    auto read_a = [&](const uint4 *st, int t) { return st[(t / 4 * 128 + wm * 64 + t % 4 * 16) * 4]; };
    auto read_b = [&](const uint4 *st, int j) { return st[(GW_ROWS + (wn * 4 + j) * 16) * 4]; };
    uint4 fa[2], fb[4];
    // the products of step kt from its stage; ends with the next step's first operands on their way into fa[0] and fb
    auto multiply = [&](int kt, bool more) {
        const uint4 *st = stage(kt), *nx = stage(kt + 1);
        uint4 nb[4];
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            if (t < 7) fa[(t + 1) & 1] = read_a(st, t + 1);
            else if (more) fa[0] = read_a(nx, 0);
            if (t == 5 && more) {
#pragma unroll
                for (int j = 0; j < 4; ++j) nb[j] = read_b(nx, j);
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) acc[t][j] = mfma_bf16(fa[t & 1], fb[j], acc[t][j]);
        }
        if (more) {
#pragma unroll
            for (int j = 0; j < 4; ++j) fb[j] = nb[j];
        }
    };
    fill(0);
    fill(1);
    fill(2);
    stage_barrier<0>();
    fa[0] = read_a(stage(0), 0);
#pragma unroll
    for (int j = 0; j < 4; ++j) fb[j] = read_b(stage(0), j);
    // at the barrier of step kt the stages kt and kt + 1 are complete, kt + 2 may be in flight
    int kt = 0;
    for (; kt + 3 < nfull; ++kt) {
        stage_barrier<4>();
        fill_full(kt + 3);                                  // into the stage that every wave has just finished with
        multiply(kt, true);
    }
    for (; kt < nk; ++kt) {
        stage_barrier<0>();
        fill(kt + 3);
        multiply(kt, kt + 1 < nk);
    }

    // the lane holds rows 4*lq .. 4*lq+3 and column lm of each 16 x 16 tile
    float *out = job.out;
    const size_t ldo = job.ldo;
    const int nl = n0 + wn * 64 + lm;
    if (pair) {
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int m = m0 + wm * 64 + t * 16 + lq * 4 + e;
                if (m >= M) continue;
                const float sc = job.scale[m];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const float z = fmaxf(acc[t][j][e], 0.f) * acc[4 + t][j][e];
                    if (nl + j * 16 < N) out[m * ldo + nl + j * 16] = z * z * sc;
                }
            }
    } else {
#pragma unroll
        for (int t = 0; t < 8; ++t)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int m = m0 + t / 4 * 128 + wm * 64 + t % 4 * 16 + lq * 4 + e;
                if (m >= M) continue;
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (nl + j * 16 < N) out[m * ldo + nl + j * 16] = acc[t][j][e];
            }
    }
}

// dst [cols][rows] = src [rows][cols]^T, 16-bit elements, 32 x 32 tiles through LDS.
__global__ __launch_bounds__(256) void k_transpose16(const uint16_t *__restrict__ src, int rows, int cols,
                                                     uint16_t *__restrict__ dst)
{
    __shared__ uint16_t tile[32][33];
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;       // 32 x 8
    const int r0 = blockIdx.y * 32, c0 = blockIdx.x * 32;
    for (int y = ty; y < 32; y += 8)
        if (r0 + y < rows && c0 + tx < cols) tile[y][tx] = src[(size_t)(r0 + y) * cols + c0 + tx];
    __syncthreads();
    for (int y = ty; y < 32; y += 8)
        if (c0 + y < cols && r0 + tx < rows) dst[(size_t)(c0 + y) * rows + r0 + tx] = tile[tx][y];
}

}   // namespace svdp
