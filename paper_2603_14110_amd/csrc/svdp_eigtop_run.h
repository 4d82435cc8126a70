// The r leading eigenvectors of a symmetric positive semi-definite matrix G [n][n] without its other n - r: a block of
// k > r vectors is filtered by Chebyshev polynomials of G that are small on [0, b], b = the block's smallest Ritz value,
// and large above (subspace iteration with Rayleigh-Ritz).  Almost all of it is k x n x n products on the fp64 matrix
// cores, about 25 of them; block Jacobi runs on the k x k projections only.  Included by svdp.hip after
// svdp_whiten_run.h's helpers, inside its unnamed namespace.
//
//   start    k pseudo-random rows, three times X <- orth(X G)
//   repeat   Rayleigh-Ritz: H = X G X^T, its eigenvectors rotate X; residuals of the wanted vectors; done if small
//            vectors that are already exact leave the block: G <- G - v theta v^T, so that a few dominant directions
//            (the mean of the tokens carries 1e8 times the energy of the rest) do not limit the filter's degree
//            X <- orth(p(G) X), as many degrees as the Ritz values say are missing, in pieces that keep X's condition
//            number below EIG_AMPLIFY
//
// Accuracy: a vector counts as found when all residuals together are below 2e-13 of ||G||_F; the Jacobi path stops at an
// off-diagonal norm of 1e-11 of it.  Rounding leaves about 1e-15.
// Measured (bf16, whole call): d = 4096, r = 256: 401 -> 50 ms (39 products of 320 x 4096 x 4096 at 0.27 ms, three
// projections of 18 Jacobi sweeps together); d = 1024, r = 64: 43.6 -> 3.8 ms; d = 2560, r = 640 (k = 832): 74 ms.
// Where it does not apply (block of more than half the dimension; no gap in reach behind the wanted vectors; X loses
// rank, e.g. G of rank below r) the full Jacobi decomposition runs instead, on the untouched G.

constexpr double EIG_TOL = 2e-13;           // sqrt(sum of squared residuals of the wanted vectors) / ||G||_F
constexpr double EIG_TOL_JACOBI = 1e-13;    // of the projected problems (off-diagonal / total Frobenius norm)
constexpr double EIG_EXACT = 2e-15;         // residual / ||G||_F below which a vector is as good as rounding allows
constexpr double EIG_AMPLIFY = 1e5;         // largest over smallest filter value between two orthogonalisations
constexpr double EIG_SHIFT = 4e-13;         // of the first Cholesky QR pass (above k_chol_diag's bound of 1e-13)

// Rows of the block for r wanted vectors: a quarter more (at least 32), so that the filter has a gap to work with, in
// whole Jacobi strips; 0 where the Jacobi decomposition of all of G is the better way.
inline int eigtop_block(int n, int r)
{
    const int k = round_up(r + std::max(32, r / 4), BJ_S);
    return 2 * k <= n ? k : 0;
}

struct EigTopWs {
    double *X, *Y, *Xa, *Xb;            // [k][n]
    double *Gd;                         // [n][n] deflated G
    double *H, *Ha, *V, *Va, *Vs, *L;   // [k][k]
    double *invL;                       // [k][64]
    double *lam, *theta, *res;          // [k]
    double *scale;                      // [1]
    double *Uall, *rowsums, *sums;      // as in WhitenWs
    double *scaled;                     // [r][n]
    int32_t *sel, *fail;
    DgScratch scr;
};

// X [k][n] becomes orthonormal by passes of Cholesky QR (Gram matrix, factor, forward substitution by blocks); the first
// pass adds EIG_SHIFT to the unit diagonal, which lets it take any condition number and leaves one that the next pass can.
// The columns' order is kept: row i stays in the span of the rows up to i.  Swaps X and tmp once per pass.
void orthonormalize(double *&X, double *&tmp, int k, int n, int passes, const EigTopWs &w, hipStream_t st)
{
    for (int p = 0; p < passes; ++p) {
        hipLaunchKernelGGL(k_normalize_rows, dim3(k), dim3(256), 0, st, X, n);
        dgemm<DG_ROWS_K, DG_ROWS_K>(op((const double *)X, n), op((const double *)X, n), w.L, k, k, k, n, st, DG_LOWER | DG_MIRROR,
                                    DgEpilogue{}, w.scr);
        if (p == 0) hipLaunchKernelGGL(k_add_diagonal, grid1(k), dim3(256), 0, st, w.L, k, EIG_SHIFT);
        cholesky_blocked(w.L, k, w.invL, w.scale, w.fail, st);
        for (int c0 = 0; c0 < k; c0 += CH_B) {
            double *done = tmp + (size_t)c0 * n, *below = X + (size_t)(c0 + CH_B) * n;
            dgemm<DG_ROWS_K, DG_K_ROWS>(op((const double *)w.invL + (size_t)c0 * CH_B, CH_B),
                                        op((const double *)X + (size_t)c0 * n, n), done, n, CH_B, n, CH_B, st);
            dgemm<DG_ROWS_K, DG_K_ROWS>(op((const double *)w.L + (size_t)(c0 + CH_B) * k + c0, k), op((const double *)done, n),
                                        below, n, k - c0 - CH_B, n, CH_B, st, 0, minus_from(below, n));
        }
        std::swap(X, tmp);
    }
}

// X <- X - (X Vl^T) Vl for the l rows of Vl
void project_out(double *X, int k, int n, const double *Vl, int l, const EigTopWs &w, hipStream_t st)
{
    if (l == 0) return;
    dgemm<DG_ROWS_K, DG_ROWS_K>(op((const double *)X, n), op(Vl, n), w.Vs, k, k, l, n, st, 0, DgEpilogue{}, w.scr);
    dgemm<DG_ROWS_K, DG_K_ROWS>(op((const double *)w.Vs, k), op(Vl, n), X, n, k, n, l, st, 0, minus_from(X, n));
}

// X <- G X (rows)
inline void times_g(const double *G, const double *X, double *out, int k, int n, hipStream_t st, const DgScratch &scr,
                    const DgEpilogue &ep = DgEpilogue{})
{
    dgemm<DG_ROWS_K, DG_ROWS_K>(op(X, n), op(G, n), out, n, k, n, n, st, 0, ep, scr);
}

// Vr [r][n] = the r leading eigenvectors of G as rows, largest eigenvalue first; lam [r] (host).  `found` = false: the
// caller takes the Jacobi decomposition (G is untouched).  sweeps: of the last projected problem.
svdp_status leading_eigenvectors(const double *G, int n, int r, double *Vr, double *lam, bool &found, int *sweeps,
                                 EigTopWs &w, hipStream_t st)
{
    found = false;
    const int k = eigtop_block(n, r);
    if (k == 0) return SVDP_OK;
    auto hip_failed = [] {
        (void)hipGetLastError();
        return SVDP_ERR_HIP;
    };
    if (hipMemsetAsync(w.fail, 0, 4, st) != hipSuccess) return hip_failed();
    std::vector<double> h(2 * (size_t)k + 2);
    double *X = w.X, *tmp = w.Xa;
    hipLaunchKernelGGL(k_random_rows, grid1((size_t)k * n), dim3(256), 0, st, X, 0, k, n);
    for (int p = 0; p < 3; ++p) {
        times_g(G, X, tmp, k, n, st, w.scr);
        std::swap(X, tmp);
        orthonormalize(X, tmp, k, n, p < 2 ? 2 : 3, w, st);
    }
    const double *Gc = G;
    double norm = 0.0, last_err = 1e300;
    int l = 0, ka = k, products = 4;             // vectors that left the block; rows of the block
    for (int cycle = 0; cycle < 12; ++cycle) {
        // Rayleigh-Ritz
        double *Y = nullptr, *Xr = nullptr, *Yr = nullptr;
        for (double *p : {w.X, w.Xa, w.Xb, w.Y})
            if (p != X) (Y == nullptr ? Y : Xr == nullptr ? Xr : Yr) = p;
        times_g(Gc, X, Y, ka, n, st, w.scr);
        dgemm<DG_ROWS_K, DG_ROWS_K>(op((const double *)X, n), op((const double *)Y, n), w.H, ka, ka, ka, n, st,
                                    DG_LOWER | DG_MIRROR, DgEpilogue{}, w.scr);
        double *A = w.H, *Aa = w.Ha, *V = w.V, *Va = w.Va;
        int sw = 0;
        const svdp_status e =
            jacobi_eigh(&A, &Aa, &V, &Va, ka, w.Uall, w.rowsums, w.sums, w.lam, EIG_TOL_JACOBI, 24, &sw, st);
        if (e != SVDP_OK) return e;
        *sweeps = std::max(1, sw);
        hipLaunchKernelGGL(k_rank_descending, grid1(ka), dim3(256), 0, st, w.lam, ka, w.sel, w.theta);
        hipLaunchKernelGGL(k_gather_rows, grid1((size_t)ka * ka), dim3(256), 0, st, V, w.sel, ka, ka, w.Vs);
        dgemm<DG_ROWS_K, DG_K_ROWS>(op((const double *)w.Vs, ka), op((const double *)X, n), Xr, n, ka, n, ka, st);
        dgemm<DG_ROWS_K, DG_K_ROWS>(op((const double *)w.Vs, ka), op((const double *)Y, n), Yr, n, ka, n, ka, st);
        hipLaunchKernelGGL(k_ritz_residual, dim3(ka), dim3(256), 0, st, Xr, Yr, w.theta, n, w.res);
        double *theta = h.data(), *res = theta + k;
        int32_t failed = 0;
        if (hipMemcpyAsync(theta, w.theta, (size_t)ka * 8, hipMemcpyDeviceToHost, st) != hipSuccess ||
            hipMemcpyAsync(res, w.res, (size_t)ka * 8, hipMemcpyDeviceToHost, st) != hipSuccess ||
            hipMemcpyAsync(&failed, w.fail, 4, hipMemcpyDeviceToHost, st) != hipSuccess ||
            hipStreamSynchronize(st) != hipSuccess)
            return hip_failed();
        X = Xr;
        if (cycle == 0) {
            // ||G||_F up to what is outside the block (which is small or else nothing here converges)
            for (int i = 0; i < ka; ++i) norm += theta[i] * theta[i];
            norm = std::sqrt(norm);
        }
        const int need = r - l;
        double err = 0.0;
        for (int i = 0; i < need; ++i) err += res[i];
        err = std::sqrt(err) / norm;
        if (failed != 0 || !(err < 1e300) || !(norm > 0.0)) return SVDP_OK;
        if (err <= EIG_TOL || (err <= 1e-12 && err > 0.5 * last_err)) {
            for (int i = 0; i < need; ++i) lam[l + i] = theta[i];
            if (hipMemcpyAsync(Vr + (size_t)l * n, X, (size_t)need * n * 8, hipMemcpyDeviceToDevice, st) != hipSuccess)
                return hip_failed();
            found = true;
            return hip_status(hipSuccess);
        }
        last_err = err;
        // degree that the Ritz values call for, with a margin for those that have not settled yet
        const double b = std::max(theta[ka - 1], 1e-15 * norm), margin = cycle == 0 ? 1e3 : 30.0;
        const double reach = std::acosh(std::max(2.0 * theta[need - 1] / b - 1.0, 1.0));
        const double degrees = std::acosh(std::max(err / EIG_TOL * margin, 2.0)) / reach;
        if (!(degrees * ka < 16.0 * n - (double)products * ka)) return SVDP_OK;       // Jacobi would be done sooner
        // exact vectors leave the block
        int out = 0;
        while (out < need && std::sqrt(res[out]) < EIG_EXACT * norm && theta[out] > 2.0 * theta[need - 1]) ++out;
        double top = theta[0];
        if (out > 0) {
            double *Vl = Vr + (size_t)l * n;
            if (hipMemcpyAsync(Vl, X, (size_t)out * n * 8, hipMemcpyDeviceToDevice, st) != hipSuccess) return hip_failed();
            hipLaunchKernelGGL(k_scale_rows, grid1((size_t)out * n), dim3(256), 0, st, Vl, w.theta, out, n, w.scaled);
            dgemm<DG_K_ROWS, DG_K_ROWS>(op((const double *)w.scaled, n), op((const double *)Vl, n), w.Gd, n, n, n, out, st,
                                        DG_LOWER | DG_MIRROR, minus_from(Gc, n));
            Gc = w.Gd;
            for (int i = 0; i < out; ++i) lam[l + i] = theta[i];
            top = theta[out];
            l += out;
            const int left = ka - out, want = std::min(k, round_up(r - l + std::max(32, r / 4), BJ_S));
            X += (size_t)out * n;                // moved to the front of a buffer by the orthonormalisation below
            double *front = Y;
            if (hipMemcpyAsync(front, X, (size_t)std::min(left, want) * n * 8, hipMemcpyDeviceToDevice, st) != hipSuccess)
                return hip_failed();
            X = front;
            if (left < want)
                hipLaunchKernelGGL(k_random_rows, grid1((size_t)(want - left) * n), dim3(256), 0, st, X, left, want - left, n);
            ka = want;
            tmp = Xr;
            for (int p = 0; p < 2; ++p) {
                hipLaunchKernelGGL(k_normalize_rows, dim3(ka), dim3(256), 0, st, X, n);
                project_out(X, ka, n, Vr, l, w, st);
                orthonormalize(X, tmp, ka, n, 1, w, st);
            }
        }
        // filter
        const double wide = std::acosh(std::max(2.0 * top / b - 1.0, 1.0));
        const int piece = (int)std::max(1.0, std::min(1000.0, std::acosh(EIG_AMPLIFY) / std::max(wide, 1e-3)));
        for (int left = (int)std::ceil(std::max(1.0, degrees)); left > 0;) {
            const int m = std::min(piece, left);
            left -= m;
            products += m;
            const double half = 0.5 * b, s0 = half / (top - half);
            double s1 = s0;
            double *prev = X, *cur = X == w.X ? w.Xa : w.X;
            DgEpilogue ep;
            ep.alpha = s1 / half;
            ep.c1 = prev;
            ep.ld1 = n;
            ep.beta = -s1;
            times_g(Gc, prev, cur, ka, n, st, w.scr, ep);
            for (int i = 2; i <= m; ++i) {
                const double s2 = 1.0 / (2.0 / s0 - s1);
                DgEpilogue e2;
                e2.alpha = 2.0 * s2 / half;
                e2.c1 = cur;
                e2.ld1 = n;
                e2.beta = -2.0 * s2;
                e2.c2 = prev;
                e2.ld2 = n;
                e2.gamma = -s1 * s2;
                times_g(Gc, cur, prev, ka, n, st, w.scr, e2);      // the new term takes the place of the one before last
                std::swap(prev, cur);
                s1 = s2;
            }
            X = cur;
            tmp = prev;
            project_out(X, ka, n, Vr, l, w, st);
            orthonormalize(X, tmp, ka, n, 2, w, st);
        }
        products += 1;
    }
    return SVDP_OK;
}
