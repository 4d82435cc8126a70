// fp64 contraction on the matrix cores for the offline build: C = alpha * A B^T + beta * C1 + gamma * C2.
//
// Bound: v_mfma_f64_16x16x4_f64 takes 64 cycles per SIMD (78.6 TFLOP/s over the chip), so a wave needs one LDS
// operand value per matrix instruction at most and what has to be kept off the critical path is the supply from
// L2: a 64 x 64 tile asks for 8.6 TB/s at full rate, a 128 x 128 tile for half of that.  Hence one kernel with the
// tile as a template parameter, two LDS stages and ONE barrier per K step (the next step's global loads are in
// flight during the products, and are stored to the other stage after them).  Operands are taken as they lie in
// memory: either [rows][K] or [K][rows], and in the storage type (bf16 and fp32 are widened on the way into LDS),
// so that neither X^T X nor (W S)^T (W S) needs a transposed or a widened copy.
// Measured at d = 4096, D = 11008, T = 8192 (bf16 inputs), before = 64 x 64 tiles, two barriers per step, 8-byte
// loads, fp64 copies of the inputs:  X^T X 7.6 -> 2.8 ms and M^T M, M [D][d] in fp64, 3.5 to 3.7 ms (lower halves: 49 and 50 to
// 53 TFLOP/s of 78.6), M = W S with the triangular 4096 x 4096 factor 3.2 ms (58 TFLOP/s); the three together 20 -> 9.6 ms.
#pragma once

#include "svdp_device.h"

namespace svdp {

typedef double f64x4_t __attribute__((ext_vector_type(4)));

__device__ __forceinline__ double as_f64(float v) { return (double)v; }
__device__ __forceinline__ double as_f64(bf16 v) { return (double)to_f32(v); }
__device__ __forceinline__ double as_f64(double v) { return v; }

// Operand as it lies in memory.  K-contiguous rows need 16-byte aligned rows; rows-contiguous operands
// additionally a row count (M or N) that is a multiple of the elements in 16 bytes.
enum DgLayout { DG_ROWS_K = 0, DG_K_ROWS = 1 };

// Parts of the product that are known to be zero or not wanted.
enum DgFlags : int {
    DG_LOWER = 1,        // only tiles that touch the lower triangle of C are formed (square tiles) ...
    DG_MIRROR = 2,       // ... and written to the upper triangle too
    DG_K_FROM_N = 4,     // B's column n is zero for k < n (a lower-triangular B given as [K][N])
    DG_K_UPTO_N = 8,     // B's row n is zero for k > n
    DG_LOOSE_A = 16,     // A (B) does not start on a 16-byte boundary: element by element
    DG_LOOSE_B = 32
};

struct DgEpilogue {
    double alpha = 1.0;
    const double *c1 = nullptr;      // may be C itself (every element is read and written by one thread)
    int ld1 = 0;
    double beta = 0.0;
    const double *c2 = nullptr;
    int ld2 = 0;
    double gamma = 0.0;
    __device__ double operator()(double acc, int m, int n) const
    {
        double v = alpha * acc;
        if (c1 != nullptr) v += beta * c1[(size_t)m * ld1 + n];
        if (c2 != nullptr) v += gamma * c2[(size_t)m * ld2 + n];
        return v;
    }
};

constexpr int DG_THREADS = 256;

template <int ROWS, int BK, DgLayout L>
struct DgStage {
    // [ROWS][BK + 2]: sixteen rows of a fragment read fall on different banks and rows stay 16-byte aligned;
    // [BK][ROWS + 16]: the four k of a fragment read alternate between the halves of the banks
    static constexpr int LD = L == DG_ROWS_K ? BK + 2 : ROWS + 16;
    static constexpr int SIZE = L == DG_ROWS_K ? ROWS * LD : BK * LD;
    static __device__ __forceinline__ int at(int row, int k) { return L == DG_ROWS_K ? row * LD + k : k * LD + row; }
};

// One operand's tile of a K step: 16-byte pieces into registers, later widened into an LDS stage.
template <typename T, int ROWS, int BK, DgLayout L>
struct DgLoader {
    static constexpr int E = 16 / sizeof(T);
    static constexpr int PIECES = ROWS * BK / E;
    static constexpr int PER = (PIECES + DG_THREADS - 1) / DG_THREADS;
    static constexpr int PPL = (L == DG_ROWS_K ? BK : ROWS) / E;      // pieces per stored line
    uint4 raw[PER];

    static __device__ __forceinline__ uint4 load(const T *__restrict__ p, bool loose)
    {
        if (!loose) return *reinterpret_cast<const uint4 *>(p);
        T v[E];
        uint4 q;
#pragma unroll
        for (int e = 0; e < E; ++e) v[e] = p[e];
        __builtin_memcpy(&q, v, 16);
        return q;
    }
    __device__ __forceinline__ void fetch(const T *__restrict__ src, int ld, int r0, int rows, int k0, int k1, bool loose)
    {
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const int id = threadIdx.x + q * DG_THREADS, line = id / PPL, c = (id % PPL) * E;
            raw[q] = make_uint4(0u, 0u, 0u, 0u);
            if (PIECES % DG_THREADS != 0 && id >= PIECES) continue;
            if (L == DG_ROWS_K) {
                if (r0 + line < rows && k0 + c < k1) raw[q] = load(src + (size_t)(r0 + line) * ld + k0 + c, loose);
            } else {
                if (k0 + line < k1 && r0 + c < rows) raw[q] = load(src + (size_t)(k0 + line) * ld + r0 + c, loose);
            }
        }
    }
    __device__ __forceinline__ void store(double *__restrict__ lds, int k0, int k1) const
    {
        using S = DgStage<ROWS, BK, L>;
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const int id = threadIdx.x + q * DG_THREADS, line = id / PPL, c = (id % PPL) * E;
            if (PIECES % DG_THREADS != 0 && id >= PIECES) continue;
            T v[E];
            __builtin_memcpy(v, &raw[q], 16);
#pragma unroll
            for (int e = 0; e < E; e += 2) {
                double2 w;
                w.x = as_f64(v[e]);
                w.y = as_f64(v[e + 1]);
                if (L == DG_ROWS_K) {                       // a piece may straddle the end of K
                    if (k0 + c + e >= k1) w.x = 0.0;
                    if (k0 + c + e + 1 >= k1) w.y = 0.0;
                }
                *reinterpret_cast<double2 *>(lds + (L == DG_ROWS_K ? S::at(line, c + e) : S::at(c + e, line))) = w;
            }
        }
    }
};

// Block tile (16 TM WM) x (16 TN WN), WM x WN = 4 waves of TM x TN matrix tiles.  Operand lanes:
// A[row = lane % 16][k = lane / 16], B likewise; register v of a result is C[4 v + lane / 16][lane % 16].
// With gridDim.z > 1 the K range is cut into parts of `kpart` and part z goes to C + z * M * ldc without the
// epilogue (k_dgemm_sum adds them in order).
template <typename TA, DgLayout LA, typename TB, DgLayout LB, int WM, int WN, int TM, int TN, int BK>
__global__ __launch_bounds__(DG_THREADS, 2) void k_dgemm(const TA *__restrict__ A, int lda, const TB *__restrict__ B, int ldb,
                                                      double *C, int ldc, int M, int N, int K, int kpart, int flags,
                                                      DgEpilogue ep)
{
    constexpr int BM = 16 * TM * WM, BN = 16 * TN * WN;
    using SA = DgStage<BM, BK, LA>;
    using SB = DgStage<BN, BK, LB>;
    extern __shared__ double dg_smem[];
    double *stA = dg_smem, *stB = dg_smem + 2 * SA::SIZE;          // two stages each
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int lm = lane & 15, lq = lane >> 4, wm = wave / WN, wn = wave % WN;
    int bm = blockIdx.y, bn = blockIdx.x;
    if (flags & DG_K_FROM_N) {                   // the longest columns of tiles first
        bm = blockIdx.x;
        bn = blockIdx.y;
    }
    if (flags & DG_LOWER) {                      // blockIdx.x counts the tiles of the lower triangle row by row
        const int t = blockIdx.x;
        bm = (int)((sqrtf(8.0f * (float)t + 1.0f) - 1.0f) * 0.5f);
        while ((bm + 1) * (bm + 2) / 2 <= t) ++bm;
        while (bm * (bm + 1) / 2 > t) --bm;
        bn = t - bm * (bm + 1) / 2;
    }
    const int m0 = bm * BM, n0 = bn * BN;
    int k_begin = blockIdx.z * kpart, k_end = min(K, k_begin + kpart);
    if (flags & DG_K_FROM_N) k_begin = max(k_begin, n0 / BK * BK);
    if (flags & DG_K_UPTO_N) k_end = min(k_end, n0 + BN);

    f64x4_t acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = f64x4_t{0.0, 0.0, 0.0, 0.0};

    const bool loose_a = sizeof(TA) < 8 && (flags & DG_LOOSE_A), loose_b = sizeof(TB) < 8 && (flags & DG_LOOSE_B);
    DgLoader<TA, BM, BK, LA> fa;
    DgLoader<TB, BN, BK, LB> fb;
    if (k_begin < k_end) {
        fa.fetch(A, lda, m0, M, k_begin, k_end, loose_a);
        fb.fetch(B, ldb, n0, N, k_begin, k_end, loose_b);
        fa.store(stA, k_begin, k_end);
        fb.store(stB, k_begin, k_end);
    }
    int cur = 0;
    for (int k0 = k_begin; k0 < k_end; k0 += BK, cur ^= 1) {
        __syncthreads();         // this step's stage is complete, the other one's readers are done
        const bool more = k0 + BK < k_end;
        if (more) {
            fa.fetch(A, lda, m0, M, k0 + BK, k_end, loose_a);
            fb.fetch(B, ldb, n0, N, k0 + BK, k_end, loose_b);
        }
        const double *pa = stA + cur * SA::SIZE, *pb = stB + cur * SB::SIZE;
#pragma unroll
        for (int kk = 0; kk < BK; kk += 4) {
            double va[TM], vb[TN];
#pragma unroll
            for (int i = 0; i < TM; ++i) va[i] = pa[SA::at((wm * TM + i) * 16 + lm, kk + lq)];
#pragma unroll
            for (int j = 0; j < TN; ++j) vb[j] = pb[SB::at((wn * TN + j) * 16 + lm, kk + lq)];
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(va[i], vb[j], acc[i][j], 0, 0, 0);
        }
        if (more) {
            fa.store(stA + (cur ^ 1) * SA::SIZE, k0 + BK, k_end);
            fb.store(stB + (cur ^ 1) * SB::SIZE, k0 + BK, k_end);
        }
    }
    const bool parts = gridDim.z > 1;
    if (parts) C += (size_t)blockIdx.z * M * ldc;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int m = m0 + (wm * TM + i) * 16 + 4 * v + lq, n = n0 + (wn * TN + j) * 16 + lm;
                // a mirrored product is symmetric to the last bit: one value for both places
                const bool mirror = (flags & DG_MIRROR) != 0;
                if (m < M && n < N && !(mirror && n > m)) {
                    const double r = parts ? acc[i][j][v] : ep(acc[i][j][v], m, n);
                    C[(size_t)m * ldc + n] = r;
                    if (mirror && n < m) C[(size_t)n * ldc + m] = r;
                }
            }
}

// C = epilogue(sum over the parts [nz][M][N], in order)
__global__ __launch_bounds__(256) void k_dgemm_sum(const double *__restrict__ parts, int nz, double *C, int ldc, int M, int N,
                                                   int flags, DgEpilogue ep)
{
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x, all = (size_t)M * N;
    if (i >= all) return;
    const int m = (int)(i / N), n = (int)(i % N);
    const size_t from = (flags & DG_MIRROR) && n > m ? (size_t)n * N + m : i;
    double s = 0.0;
    for (int z = 0; z < nz; ++z) s += parts[(size_t)z * all + from];
    C[(size_t)m * ldc + n] = ep(s, m, n);
}

}   // namespace svdp
