// Host side of the offline build with whitening (Alg. 1): fp64 work buffers, the launches of the contraction kernel
// and the drivers of the factorisations.  Included by svdp.hip inside its unnamed namespace.

inline dim3 grid1(size_t n) { return dim3((unsigned)((n + 255) / 256)); }

// ---- C = alpha A B^T + beta C1 + gamma C2 (k_dgemm): operands and the choice of the tile ----

template <typename T>
struct DgOperand {
    const T *p;
    int ld;
};
template <typename T>
DgOperand<T> op(const T *p, int ld) { return DgOperand<T>{p, ld}; }

struct DgScratch {          // where parts of a split K range meet
    double *p;
    size_t n;               // doubles
};

template <typename TA, DgLayout LA, typename TB, DgLayout LB, int WM, int WN, int TM, int TN, int BK>
[[nodiscard]] bool dgemm_tile(DgOperand<TA> A, DgOperand<TB> B, double *C, int ldc, int M, int N, int K, int flags, const DgEpilogue &ep,
                int nz, const DgScratch &scr, hipStream_t st)
{
    constexpr int BM = 16 * TM * WM, BN = 16 * TN * WN;
    constexpr auto kernel = &k_dgemm<TA, LA, TB, LB, WM, WN, TM, TN, BK>;
    constexpr size_t lds = (size_t)2 * (DgStage<BM, BK, LA>::SIZE + DgStage<BN, BK, LB>::SIZE) * 8;
    if (!grant_lds<kernel>(lds)) return false;
    const int tm = (M + BM - 1) / BM, tn = (N + BN - 1) / BN;
    int kpart = K;
    if (nz > 1) {
        kpart = round_up((K + nz - 1) / nz, BK);
        nz = (K + kpart - 1) / kpart;
    }
    const dim3 grid = (flags & DG_LOWER) ? dim3(tm * (tm + 1) / 2, 1, nz)
                                         : (flags & DG_K_FROM_N) ? dim3(tm, tn, nz) : dim3(tn, tm, nz);
    if (nz > 1) {
        launch(kernel, grid, dim3(DG_THREADS), lds, st, A.p, A.ld, B.p, B.ld, scr.p, N, M, N, K, kpart, flags,
               DgEpilogue{});
        launch(k_dgemm_sum, grid1((size_t)M * N), dim3(256), 0, st, scr.p, nz, C, ldc, M, N, flags, ep);
    } else {
        launch(kernel, grid, dim3(DG_THREADS), lds, st, A.p, A.ld, B.p, B.ld, C, ldc, M, N, K, kpart, flags, ep);
    }
    return true;
}

// Tile and split of a product.  false: the device does not grant the LDS a tile needs, nothing was enqueued (every function
// that forms products hands this on, and the call answers SVDP_ERR_UNSUPPORTED).  DG_LOWER needs M == N.  `one_tile_wide` (N <= 64): every block covers all columns of
// its rows, so that C may be A itself.
//  - large products: 128 x 128, 96 x 96 or 64 x 64 tiles, whichever leaves the least idle in the last round (the lower
//    half of a 4096 x 4096 product is 528 tiles of 128 x 128, i.e. 2.06 rounds of the 256 compute units that take the
//    time of three, but 946 of 96 x 96, 3.7 rounds of 9/16 of the work each); a smaller tile reads more from L2 per
//    product, which the weights stand for;
//  - 80 x 64 tiles (four waves side by side) likewise: 320 rows by 4096 columns are exactly 256 of them;
//  - small products: 32 x 32 tiles and parts of K (k_dgemm_sum adds them in order).
template <DgLayout LA, DgLayout LB, typename TA, typename TB>
[[nodiscard]] bool dgemm(DgOperand<TA> A, DgOperand<TB> B, double *C, int ldc, int M, int N, int K, hipStream_t st, int flags = 0,
           const DgEpilogue &ep = DgEpilogue{}, const DgScratch &scr = DgScratch{nullptr, 0}, bool one_tile_wide = false)
{
    if (M <= 0 || N <= 0) return true;
    if (!aligned16(A.p)) flags |= DG_LOOSE_A;       // possible for the caller's own matrices only
    if (!aligned16(B.p)) flags |= DG_LOOSE_B;
    auto tiles = [&](int bm, int bn) {
        const long long tm = (M + bm - 1) / bm, tn = (N + bn - 1) / bn;
        return (flags & DG_LOWER) ? tm * (tm + 1) / 2 : tm * tn;
    };
    constexpr long long CUS = 256;
    if (one_tile_wide) return dgemm_tile<TA, LA, TB, LB, 2, 2, 2, 2, 16>(A, B, C, ldc, M, N, K, flags, ep, 1, scr, st);
    if (tiles(64, 64) >= 200) {
        auto cost = [&](int bm, int bn, double weight) {
            return (double)((tiles(bm, bn) + CUS - 1) / CUS) * bm * bn * weight;
        };
        const bool lower = (flags & DG_LOWER) != 0;
        const double c128 = cost(128, 128, 1.0), c96 = cost(96, 96, 1.05), c64 = cost(64, 64, 1.25),
                     c80 = lower ? 1e300 : cost(80, 64, 1.2);
        const double best = std::min(std::min(c128, c96), std::min(c64, c80));
        // at most one block per compute unit has nobody to hide its loads and barriers behind: two parts of K
        // (256 x 4096 x 4096: 250 -> 160 us with the sum)
        const auto parts = [&](int bm, int bn) { return tiles(bm, bn) <= CUS && K >= 1024 && (size_t)2 * M * N <= scr.n ? 2 : 1; };
        if (best == c128)
            return dgemm_tile<TA, LA, TB, LB, 2, 2, 4, 4, 16>(A, B, C, ldc, M, N, K, flags, ep, parts(128, 128), scr, st);
        if (best == c96) return dgemm_tile<TA, LA, TB, LB, 2, 2, 3, 3, 16>(A, B, C, ldc, M, N, K, flags, ep, parts(96, 96), scr, st);
        if (best == c80) return dgemm_tile<TA, LA, TB, LB, 1, 4, 5, 1, 32>(A, B, C, ldc, M, N, K, flags, ep, parts(80, 64), scr, st);
        return dgemm_tile<TA, LA, TB, LB, 2, 2, 2, 2, 16>(A, B, C, ldc, M, N, K, flags, ep, parts(64, 64), scr, st);
    }
    const long long t32 = tiles(32, 32);
    int nz = (int)std::max<long long>(1, std::min<long long>(2 * CUS / t32, K / 256));
    while (nz > 1 && (size_t)nz * M * N > scr.n) --nz;
    return dgemm_tile<TA, LA, TB, LB, 2, 2, 1, 1, 32>(A, B, C, ldc, M, N, K, flags, ep, nz, scr, st);
}

// C = Cin - (product)
inline DgEpilogue minus_from(const double *Cin, int ld)
{
    DgEpilogue e;
    e.alpha = -1.0;
    e.c1 = Cin;
    e.ld1 = ld;
    e.beta = 1.0;
    return e;
}

// The lower triangle of A [n][n] (n a multiple of 64) becomes L with L L^T = A, zero above the diagonal; invL:
// [n/64][64][64], the inverses of L's diagonal blocks; scale: device double; fail: device int, set to 1 if A is not
// positive definite to working precision (then L is not to be used).
[[nodiscard]] bool cholesky_blocked(double *A, int n, double *invL, double *scale, int *fail, hipStream_t st)
{
    bool ok = true;
    launch(k_max_diag, dim3(1), dim3(256), 0, st, A, n, scale);
    for (int k = 0; k < n; k += CH_B) {
        const int p1 = std::min(n, k / CH_PANEL * CH_PANEL + CH_PANEL);       // end of the panel
        const int k1 = k + CH_B, rest = n - k1;
        double *inv = invL + (size_t)k * CH_B;
        launch(k_chol_diag, dim3(1), dim3(256), 0, st, A, n, (size_t)k * n + k, scale, 1e-13, inv, fail);
        const double *below = A + (size_t)k1 * n + k;
        // in place: a block of the product covers all 64 columns of its rows
        ok &= dgemm<DG_ROWS_K, DG_ROWS_K>(op(below, n), op((const double *)inv, CH_B), A + (size_t)k1 * n + k, n, rest, CH_B,
                                          CH_B, st, 0, DgEpilogue{}, DgScratch{nullptr, 0}, true);
        double *upd = A + (size_t)k1 * n + k1;
        ok &= dgemm<DG_ROWS_K, DG_ROWS_K>(op(below, n), op(below, n), upd, n, rest, p1 - k1, CH_B, st, 0, minus_from(upd, n));
        if (k1 == p1 && rest > 0) {
            const double *pan = A + (size_t)k1 * n + (k1 / CH_PANEL - 1) * CH_PANEL;
            ok &= dgemm<DG_ROWS_K, DG_ROWS_K>(op(pan, n), op(pan, n), upd, n, rest, rest, CH_PANEL, st, DG_LOWER,
                                              minus_from(upd, n));
        }
    }
    launch(k_zero_upper_blocks, grid1((size_t)n * n), dim3(256), 0, st, A, n);
    return ok;
}

// Bout [r][n] = Bin [r][n] L^-1 for the lower-triangular L [n][n] and the inverses of its diagonal blocks: block
// back-substitution from the last block column to the first.  A finished block column is taken out of all columns to
// its left at once (a wide product with K = 64).  Bin is destroyed.
[[nodiscard]] bool solve_right_lower(double *Bin, double *Bout, int r, int n, const double *L, const double *invL, hipStream_t st)
{
    bool ok = true;
    for (int c0 = n - CH_B; c0 >= 0; c0 -= CH_B) {
        ok &= dgemm<DG_ROWS_K, DG_K_ROWS>(op((const double *)Bin + c0, n), op(invL + (size_t)c0 * CH_B, CH_B), Bout + c0, n, r,
                                          CH_B, CH_B, st);
        ok &= dgemm<DG_ROWS_K, DG_K_ROWS>(op((const double *)Bout + c0, n), op(L + (size_t)c0 * n, n), Bin, n, r, c0, CH_B, st, 0,
                                          minus_from(Bin, n));
    }
    return ok;
}

// Eigen-decomposition of the symmetric matrix in *A (n x n, n % 64 == 0) by block Jacobi sweeps.  On return
// *A / *V point at the buffers holding the (numerically) diagonal matrix and the eigenvectors as rows, lam[i]
// (device) = (*A)[i][i].  Uall: n/64 matrices of 64 x 64.  Synchronises the stream once per sweep (the
// convergence figure is read on the host).
svdp_status jacobi_eigh(double **A, double **Aalt, double **V, double **Valt, int n, double *Uall, double *rowsums,
                        double *sums, double *lam, double tol, int max_sweeps, int *sweeps_out, hipStream_t st)
{
    const size_t lds_solve = BJ_SOLVE_LDS, lds_apply = (size_t)2 * BJ_S * BJ_LD * 8;
    if (!grant_lds<k_bjacobi_solve<false>>(lds_solve) || !grant_lds<k_bjacobi_solve<true>>(lds_solve) ||
        !grant_lds<k_bjacobi_apply>(lds_apply))
        return SVDP_ERR_UNSUPPORTED;
    launch(k_identity, grid1((size_t)n * n), dim3(256), 0, st, *V, n);
    const int strips = n / BJ_S, rounds = n / BJ_B > 2 ? n / BJ_B - 1 : 1;
    const int ct = strips >= 32 ? 4 : 1, cgrid = (strips + ct - 1) / ct;      // column tiles per block
    double previous = 1e300;
    int sweep = 0;
    for (;; ++sweep) {
        launch(k_jacobi_norms, dim3(n), dim3(256), 0, st, *A, n, rowsums);
        launch(k_jacobi_norms_finish, dim3(1), dim3(256), 0, st, rowsums, n, *A, sums, lam);
        double h[2] = {0.0, 0.0};
        if (hipMemcpyAsync(h, sums, sizeof(h), hipMemcpyDeviceToHost, st) != hipSuccess ||
            hipStreamSynchronize(st) != hipSuccess) {
            (void)hipGetLastError();
            return SVDP_ERR_HIP;
        }
        // a tolerance near rounding may not be reached: below 1e-11, where the whole matrix is taken as diagonal, a sweep
        // that gains less than a factor of two is the last
        const bool stalled = h[0] <= 1e-22 * h[1] && h[0] > 0.25 * previous;
        if (!(h[1] == h[1]) || h[0] <= tol * tol * h[1] || stalled || sweep >= max_sweeps) break;
        previous = h[0];
        for (int round = 0; round < rounds; ++round) {
            // A sweep's first round takes the pairs inside the blocks as well, which all have their turn in it; the others only
            // those across: half the steps, and a sweep or two more.  With few rounds the first sweep is worth having whole.
            // Whole call, every round whole / this (ms): n = 512, r = 400 (full decomposition) 11.8 / 7.6, d = 2560, r = 640
            // 53.3 / 48.9, d = 4096, r = 256 42.5 / 40.3, d = 1024, r = 64 4.2 / 3.1; without the first sweep at d = 320,
            // r = 80 4.4 / 4.5, with it 4.35.
            if (round == 0 || (sweep == 0 && rounds <= 5))
                launch(k_bjacobi_solve<false>, dim3(strips, BJ_U_PARTS), dim3(BJ_SOLVE_THREADS), lds_solve, st, *A, n, Uall);
            else
                launch(k_bjacobi_solve<true>, dim3(strips, BJ_U_PARTS), dim3(BJ_SOLVE_THREADS), lds_solve, st, *A, n, Uall);
            launch(k_bjacobi_apply, dim3(cgrid, strips, 2), dim3(256), lds_apply, st, *A, *V, Uall, n, ct, *Aalt, *Valt);
            std::swap(*A, *Aalt);
            std::swap(*V, *Valt);
        }
    }
    if (sweeps_out != nullptr) *sweeps_out = sweep;
    return hip_status(hipSuccess);
}
