// The r leading eigenvectors of G = M^T M [n][n] without its other n - r: a block of k > r vectors is filtered by Chebyshev
// polynomials of G that are small on [0, b], b = the block's smallest Ritz value, and large above (subspace iteration with
// Rayleigh-Ritz).  Almost all of it is k x n x n products on the fp64 matrix cores, 4 to 50 of them; block Jacobi runs on the
// k x k projections only.  Included by svdp.hip after svdp_whiten_run.h's helpers, inside its unnamed namespace.
//
//   start    k pseudo-random rows, three times X <- orth(X G)
//   repeat   Rayleigh-Ritz: H = X G X^T, its eigenvectors rotate X; residuals of the wanted vectors; done if small
//            dominant vectors that have settled leave the block: M <- M - (M v) v^T and G is formed again
//            X <- orth(p(G) X), as many degrees as the Ritz values say are missing, in pieces of at most EIG_PIECE that
//            also keep X's condition number below EIG_AMPLIFY
//
// Accuracy: a stored G, and every product with it, carries an error of a few 2^-53 of its LARGEST eigenvalue.  The mean of the
// tokens alone often has 1e8 times the energy of the wanted directions behind it, so that error and a residual measured
// against ||G|| say nothing about those.  Hence what dominates is taken out of the factor M, whose elements only carry 2^-53
// of the largest singular value, until the block's eigenvalues are within EIG_SPREAD of each other; and the residuals of
// the wanted vectors together end below EIG_TOL (where they stop falling first: 5 EIG_TOL) of the SMALLEST wanted eigenvalue.
// Against singular values worked out with 64-bit mantissas (d = 256, r = 40, tokens with a mean of 10 to 3e6 times their
// spread; geometric spectra over up to twelve decades): within 4e-12 each, the product within 2e-9 of sigma_r.
// Measured (bf16, 64 dominant directions, whole call), full Jacobi -> this: d = 4096, r = 256: 311 -> 39.5 ms (56 products of 256
// to 320 x 4096 x 4096 at 0.16 to 0.22 ms, two projections, G once more); d = 1024, r = 64: 24 -> 2.9 ms; d = 2560, r = 640:
// 105 -> 46 ms.  With b fixed between projections and pieces as long as the condition number allowed, the
// first took three projections: b starts at 0.65 of where it ends, which costs three quarters of the filter's rate.  With
// EIG_SETTLED = 1e-13 a projection more was needed at d = 512, r = 128 (9.1 against 6.2 ms): vectors that share a strip of the
// projected matrix with the largest are left with that much.
// Where it does not apply (block of more than half the dimension; no gap in reach behind the wanted vectors; fewer than r
// singular values above rounding) the full Jacobi decomposition runs instead, on the untouched G.

// sqrt(sum of squared residuals of the wanted vectors) / smallest wanted eigenvalue: a vector whose eigenvalue is a
// thousandth away from the first unwanted one is then off by 2e-8, which fp32 results do not show
constexpr double EIG_TOL = 2e-11;
constexpr double EIG_TOL_JACOBI = 1e-12;    // of the projected problems (off-diagonal / total Frobenius norm), or less where
                                            // the wanted eigenvalues are small in them
// Largest over smallest eigenvalue of one block.  Up to here the error of G, 1e-16 of the largest, is 1e-13 of the smallest.
constexpr double EIG_SPREAD = 1e3;
constexpr double EIG_SETTLED = 5e-13;       // residual of a vector that may leave, of sqrt(its eigenvalue * the largest)
constexpr double EIG_NOISE = 2e-28;         // eigenvalues below this part of the largest are rounding errors of M
constexpr double EIG_AMPLIFY = 1e5;         // largest over smallest filter value between two orthogonalisations
constexpr double EIG_PIECE = 8.0;           // largest degree of a piece of the filter
constexpr double EIG_SHIFT = 4e-13;         // of the first Cholesky QR pass (above k_chol_diag's bound of 1e-13)

// Rows of the block for r wanted vectors: a quarter more (at least 32), so that the filter has a gap to work with, in
// whole Jacobi strips; 0 where the Jacobi decomposition of all of G is the better way.  Whole call in ms, this / full, for random
// weights and tokens with a mean of 0, 10, 1e4 times their spread, weights with squared singular values 10^(-6 i / r), exp(-i / d),
// 1 / (1 + i), and a gate matrix of 64 dominant directions with correlated tokens:
//   d = 256, r = 64    3.8 / 3.8    5.2 / 3.5    4.2 / 3.1    3.3 / 8.8    3.9 / 3.4    5.4 / 3.7    4.0 / 4.5
//   d = 512, r = 64    4.4 / 7.5    6.1 / 7.5    4.7 / 6.8    2.4 / 17     4.5 / 7.3    6.3 / 8.0    3.6 / 9.6
//   d = 512, r = 200   8.3 / 7.5     12 / 7.4    8.9 / 6.8    6.5 / 17     8.2 / 7.3     16 / 7.9    8.8 / 9.6
//   d = 1024, r = 256   12 / 18      20 / 18      13 / 16      12 / 37      12 / 17      20 / 19      11 / 24
//   d = 1024, r = 400   18 / 18      31 / 18      19 / 16      13 / 37      18 / 17      31 / 19      20 / 24
// The largest block (k = n / 2) is level on flat spectra, loses where a mean or a head of some ten to a hundred times the rest asks
// for a second projection, and wins where the spectrum decays, on which the full decomposition takes all of its 24 sweeps: in
// these, at most 2.0 times slower and up to 2.8 times faster, and which of the two is known after a projection, half of its
// time.  At k = n / 3 it is behind on some (d = 384, r = 96 flat 6.2 / 5.5, 1 / (1 + i) 8.8 / 5.7), at n / 4 level or ahead on all.
// At n = 128 it is behind on all but decaying spectra (r = 16: 2.0 / 1.8 flat, 2.8 / 1.8 with a mean of 10, 1.4 / 3.9 on
// 10^(-6 i / r)).
inline int eigtop_block(int n, int r)
{
    const int k = round_up(r + std::max(32, r / 4), BJ_S);
    return n >= 256 && 2 * k <= n ? k : 0;
}

// Rough times (us) of what the iteration and the full decomposition consist of, fitted to n = 256 .. 4096: a product of k
// rows with G, one orthonormalisation, `sweeps` Jacobi sweeps over an m x m matrix.  The iteration goes on while what it
// still needs is below the full decomposition's 14 sweeps (it takes 8 to 12 on flat spectra, 12 to 15 behind 64 dominant
// directions, 24 on strongly decaying ones), and while it has not spent one and a half times as much.  Nine or eleven sweeps
// there end it just before it is done: d = 512, r = 200 and a mean of 10: 11.8 -> 16.6 / 11.8 ms, 1 / (1 + i): 15.7 -> 17.1 / 20.7;
// d = 1024, r = 400: 31 -> 44 / 44, 30 -> 40 / 45; no case gains.
// Tried: handing over after the first projection where the pieces are short (a second one will be needed): d = 1024, r = 400 and
// a mean of 10 31 -> 26, 1 / (1 + i) 30 -> 27, but d = 512, r = 128 and a mean of 10 9.7 -> 10.6, d = 256, r = 64 and a mean of 3
// 4.0 -> 5.6.  A limit on products alone (16 n rows) left out that at k = n / 2 the projections and orthonormalisations are
// most of the time, and gave up blocks that were three products short.
inline double eig_product_us(int k, int n) { return 6.0 + 5e-8 * k * (double)n * n; }
inline double eig_orthonormalize_us(int k) { return 40.0 + 0.8 * k; }
inline double eig_jacobi_us(int m, int sweeps) { return sweeps * (m / BJ_B - 1) * (40.0 + 9e-6 * m * (double)m); }

struct EigTopWs {
    int k;                              // eigtop_block(n, r)
    double *X, *Y, *Xa, *Xb;            // [k][n]
    double *M;                          // [D][n], G = M^T M; what leaves the block is taken out of it
    int D;
    double *MV;                         // [D][<= r]
    double *Gd;                         // [n][n] G formed again
    double *H, *Ha, *V, *Va, *Vs, *L;   // [k][k]
    double *invL;                       // [k][64]
    double *lam, *theta, *res;          // [k]
    double *scale;                      // [1]
    double *Uall, *rowsums, *sums;      // as in WhitenWs
    int32_t *sel, *fail;
    DgScratch scr;
};

// X [k][n] becomes orthonormal by passes of Cholesky QR (Gram matrix, factor, forward substitution by blocks); the first
// pass adds EIG_SHIFT to the unit diagonal, which lets it take any condition number and leaves one that the next pass can.
// The columns' order is kept: row i stays in the span of the rows up to i.  Swaps X and tmp once per pass.
[[nodiscard]] bool orthonormalize(double *&X, double *&tmp, int k, int n, int passes, const EigTopWs &w, hipStream_t st)
{
    bool ok = true;
    for (int p = 0; p < passes; ++p) {
        launch(k_normalize_rows, dim3(k), dim3(256), 0, st, X, n);
        ok &= dgemm<DG_ROWS_K, DG_ROWS_K>(op((const double *)X, n), op((const double *)X, n), w.L, k, k, k, n, st,
                                          DG_LOWER | DG_MIRROR, DgEpilogue{}, w.scr);
        if (p == 0) launch(k_add_diagonal, grid1(k), dim3(256), 0, st, w.L, k, EIG_SHIFT);
        ok &= cholesky_blocked(w.L, k, w.invL, w.scale, w.fail, st);
        for (int c0 = 0; c0 < k; c0 += CH_B) {
            double *done = tmp + (size_t)c0 * n, *below = X + (size_t)(c0 + CH_B) * n;
            ok &= dgemm<DG_ROWS_K, DG_K_ROWS>(op((const double *)w.invL + (size_t)c0 * CH_B, CH_B),
                                              op((const double *)X + (size_t)c0 * n, n), done, n, CH_B, n, CH_B, st);
            ok &= dgemm<DG_ROWS_K, DG_K_ROWS>(op((const double *)w.L + (size_t)(c0 + CH_B) * k + c0, k),
                                              op((const double *)done, n), below, n, k - c0 - CH_B, n, CH_B, st, 0,
                                              minus_from(below, n));
        }
        std::swap(X, tmp);
    }
    return ok;
}

// X <- X - (X Vl^T) Vl for the l rows of Vl and the ka of X.  The coefficients lie in Vs with the full block's stride: as
// vectors leave the block, l outgrows ka, but never w.k (l < r < w.k).
[[nodiscard]] bool project_out(double *X, int ka, int n, const double *Vl, int l, const EigTopWs &w, hipStream_t st)
{
    if (l == 0) return true;
    if (l > w.k || ka > w.k) return false;
    return dgemm<DG_ROWS_K, DG_ROWS_K>(op((const double *)X, n), op(Vl, n), w.Vs, w.k, ka, l, n, st, 0, DgEpilogue{}, w.scr) &&
           dgemm<DG_ROWS_K, DG_K_ROWS>(op((const double *)w.Vs, w.k), op(Vl, n), X, n, ka, n, l, st, 0, minus_from(X, n));
}

// X <- G X (rows)
[[nodiscard]] inline bool times_g(const double *G, const double *X, double *out, int k, int n, hipStream_t st,
                                  const DgScratch &scr, const DgEpilogue &ep = DgEpilogue{})
{
    return dgemm<DG_ROWS_K, DG_ROWS_K>(op(X, n), op(G, n), out, n, k, n, n, st, 0, ep, scr);
}

// M <- M - (M Vl^T) Vl for the l rows of Vl, l < r
[[nodiscard]] bool take_out_of_factor(const double *Vl, int l, int n, const EigTopWs &w, hipStream_t st)
{
    const int ld = l + (l & 1);                                // 16-byte aligned rows
    return dgemm<DG_ROWS_K, DG_ROWS_K>(op((const double *)w.M, n), op(Vl, n), w.MV, ld, w.D, l, n, st, 0, DgEpilogue{}, w.scr) &&
           dgemm<DG_ROWS_K, DG_K_ROWS>(op((const double *)w.MV, ld), op(Vl, n), w.M, n, w.D, n, l, st, 0, minus_from(w.M, n));
}

// Vr [r][n] = the r leading eigenvectors of G = M^T M as rows, largest eigenvalue first; lam [r] (host).  M is destroyed.
// `found` = false: the caller takes the Jacobi decomposition (G is untouched).  sweeps: of the last projected problem.
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
    bool ok = true;                                         // every product so far was enqueued
    double *X = w.X, *tmp = w.Xa;
    launch(k_random_rows, grid1((size_t)k * n), dim3(256), 0, st, X, 0, k, n);
    for (int p = 0; p < 3; ++p) {
        ok &= times_g(G, X, tmp, k, n, st, w.scr);
        std::swap(X, tmp);
        ok &= orthonormalize(X, tmp, k, n, p < 2 ? 1 : 3, w, st);
    }
    const double *Gc = G;
    double largest = 0.0, last_err = 1e300, jacobi_tol = EIG_TOL_JACOBI;
    const double full = eig_jacobi_us(n, 14);
    double spent = 3.0 * eig_product_us(k, n) + 5.0 * eig_orthonormalize_us(k);        // us so far, roughly
    int l = 0, ka = k, piece = 0;                           // vectors that left the block; rows of the block
    for (int cycle = 0; cycle < 24; ++cycle) {
        // Rayleigh-Ritz
        double *Y = nullptr, *Xr = nullptr, *Yr = nullptr;
        for (double *p : {w.X, w.Xa, w.Xb, w.Y})
            if (p != X) (Y == nullptr ? Y : Xr == nullptr ? Xr : Yr) = p;
        ok &= times_g(Gc, X, Y, ka, n, st, w.scr);
        ok &= dgemm<DG_ROWS_K, DG_ROWS_K>(op((const double *)X, n), op((const double *)Y, n), w.H, ka, ka, ka, n, st,
                                    DG_LOWER | DG_MIRROR, DgEpilogue{}, w.scr);
        double *A = w.H, *Aa = w.Ha, *V = w.V, *Va = w.Va;
        int sw = 0;
        const svdp_status e =
            jacobi_eigh(&A, &Aa, &V, &Va, ka, w.Uall, w.rowsums, w.sums, w.lam, jacobi_tol, 24, &sw, st);
        if (e != SVDP_OK) return e;
        *sweeps = std::max(1, sw);
        spent += 3.0 * eig_product_us(ka, n) + eig_jacobi_us(ka, sw);
        launch(k_rank_descending, grid1(ka), dim3(256), 0, st, w.lam, ka, w.sel, w.theta);
        launch(k_gather_rows, grid1((size_t)ka * ka), dim3(256), 0, st, V, w.sel, ka, ka, w.Vs);
        ok &= dgemm<DG_ROWS_K, DG_K_ROWS>(op((const double *)w.Vs, ka), op((const double *)X, n), Xr, n, ka, n, ka, st);
        ok &= dgemm<DG_ROWS_K, DG_K_ROWS>(op((const double *)w.Vs, ka), op((const double *)Y, n), Yr, n, ka, n, ka, st);
        launch(k_ritz_residual, dim3(ka), dim3(256), 0, st, Xr, Yr, w.theta, n, w.res);
        if (!ok) return SVDP_ERR_UNSUPPORTED;
        double *theta = h.data(), *res = theta + k;
        int32_t failed = 0;
        if (hipMemcpyAsync(theta, w.theta, (size_t)ka * 8, hipMemcpyDeviceToHost, st) != hipSuccess ||
            hipMemcpyAsync(res, w.res, (size_t)ka * 8, hipMemcpyDeviceToHost, st) != hipSuccess ||
            hipMemcpyAsync(&failed, w.fail, 4, hipMemcpyDeviceToHost, st) != hipSuccess ||
            hipStreamSynchronize(st) != hipSuccess)
            return hip_failed();
        X = Xr;
        if (cycle == 0) largest = theta[0];
        const int need = r - l;
        const double smallest = theta[ka - 1], tol = EIG_TOL * theta[need - 1];
        double err = 0.0;
        for (int i = 0; i < need; ++i) err += res[i];
        err = std::sqrt(err);
        if (failed != 0 || !(err < 1e300) || !(theta[0] > EIG_NOISE * largest)) return SVDP_OK;
        if (theta[0] <= EIG_SPREAD * theta[need - 1] && (err <= tol || (err <= 5.0 * tol && err > 0.5 * last_err))) {
            for (int i = 0; i < need; ++i) lam[l + i] = theta[i];
            if (hipMemcpyAsync(Vr + (size_t)l * n, X, (size_t)need * n * 8, hipMemcpyDeviceToDevice, st) != hipSuccess)
                return hip_failed();
            found = true;
            return hip_status(hipSuccess);
        }
        last_err = err;
        // Settled vectors leave the block, the largest first and not beyond EIG_SPREAD.  What is left of their residual couples
        // them to the rest of G by as little, far below the filter's edge, so it does not grow.
        double wanted = theta[need - 1], margin = 10.0;
        int out = 0;
        while (out + 1 < need && theta[out] > 2.0 * wanted && theta[out] * EIG_SPREAD >= theta[0] &&
               std::sqrt(res[out]) < EIG_SETTLED * std::sqrt(theta[0] * theta[out]))
            ++out;
        double rest = 0.0;
        for (int i = out; i < ka; ++i) rest += theta[i] * theta[i];
        jacobi_tol = std::max(1e-15, std::min(EIG_TOL_JACOBI, 0.25 * tol / std::sqrt(rest)));
        if (out > 0) {
            double *Vl = Vr + (size_t)l * n;
            if (hipMemcpyAsync(Vl, X, (size_t)out * n * 8, hipMemcpyDeviceToDevice, st) != hipSuccess) return hip_failed();
            for (int i = 0; i < out; ++i) lam[l + i] = theta[i];
            l += out;
            // the second time all of them: the first leaves 2^-53 of what was taken out, which may be more than the rest
            ok &= take_out_of_factor(Vl, out, n, w, st);
            ok &= take_out_of_factor(Vr, l, n, w, st);
            ok &= dgemm<DG_K_ROWS, DG_K_ROWS>(op((const double *)w.M, n), op((const double *)w.M, n), w.Gd, n, n, n, w.D, st,
                                        DG_LOWER | DG_MIRROR, DgEpilogue{}, w.scr);
            Gc = w.Gd;
            spent += eig_product_us(w.D / 2, n) + 3.0 * eig_orthonormalize_us(ka);
            const int left = ka - out, want = std::min(k, round_up(r - l + std::max(32, r / 4), BJ_S));
            X += (size_t)out * n;                // moved to the front of a buffer by the orthonormalisation below
            double *front = Y;
            if (hipMemcpyAsync(front, X, (size_t)std::min(left, want) * n * 8, hipMemcpyDeviceToDevice, st) != hipSuccess)
                return hip_failed();
            X = front;
            if (left < want)
                launch(k_random_rows, grid1((size_t)(want - left) * n), dim3(256), 0, st, X, left, want - left, n);
            ka = want;
            tmp = Xr;
            for (int p = 0; p < 2; ++p) {
                launch(k_normalize_rows, dim3(ka), dim3(256), 0, st, X, n);
                ok &= project_out(X, ka, n, Vr, l, w, st);
                ok &= orthonormalize(X, tmp, ka, n, p + 1, w, st);
            }
            last_err = 1e300;
            margin = 100.0;                      // the residuals were those of the old G; another projection costs more
            if (!(wanted > 1e-14 * theta[0])) continue;        // the Ritz values behind them were rounding errors
        }
        if (!(wanted > 0.0)) return SVDP_OK;
        const double top = theta[out];
        // Filter, in pieces.  Before each but the first, b follows the smallest Rayleigh quotient of the block, which is
        // near its smallest Ritz value (the rows stay in the order of the Ritz values): it rises while the block's last rows
        // settle, and the rate hangs on it, because what lies outside the block is only damped as far as b reaches.
        double bound = std::max(smallest, 1e-15 * top), todo = std::log(std::max(err / tol * margin, 2.0));
        auto growth = [](double value, double edge) { return std::acosh(std::max(2.0 * value / edge - 1.0, 1.0)); };
        int single = 0;
        for (bool first = true, last = false; !last; first = false) {
            double *prev = X, *cur = X == w.X ? w.Xa : w.X;
            if (!first) {
                ok &= times_g(Gc, X, cur, ka, n, st, w.scr);
                if (!ok) return SVDP_ERR_UNSUPPORTED;
                launch(k_rayleigh, dim3(ka), dim3(256), 0, st, X, cur, n, w.res);
                if (hipMemcpyAsync(res, w.res, (size_t)ka * 8, hipMemcpyDeviceToHost, st) != hipSuccess ||
                    hipStreamSynchronize(st) != hipSuccess)
                    return hip_failed();
                std::sort(res, res + ka, std::greater<double>());
                const double lowest = res[ka - 1];
                wanted = std::max(wanted, res[r - l - 1]);         // has risen, too
                if (!(lowest < wanted)) return SVDP_OK;            // no gap at all (also NaN)
                // what the last piece gained where the new bound now is
                todo += piece * growth(lowest, bound);
                bound = std::max(bound, lowest);
            }
            const double rate = growth(wanted, bound), left = std::ceil(todo / rate);
            // no gap in reach: the full decomposition would be done sooner
            const double pass = eig_orthonormalize_us(ka),
                         missing = left * (eig_product_us(ka, n) + pass / EIG_PIECE) + pass + eig_jacobi_us(ka, 4);
            if (!(missing < full && spent < 1.5 * full)) return SVDP_OK;
            piece = (int)std::max(1.0, std::min({EIG_PIECE, std::floor(std::acosh(EIG_AMPLIFY) / std::max(growth(top, bound), 1e-3)), left}));
            last = piece >= left || (piece == 1 && ++single == 3);  // a dominant direction keeps the pieces short: project, it may have settled
            todo -= piece * rate;
            spent += piece * eig_product_us(ka, n) + pass;
            const double half = 0.5 * bound, s0 = half / (top - half);
            double s1 = s0;
            DgEpilogue ep;
            ep.alpha = s1 / half;
            ep.c1 = prev;
            ep.ld1 = n;
            ep.beta = -s1;
            if (first) ok &= times_g(Gc, prev, cur, ka, n, st, w.scr, ep);
            else launch(k_combine, grid1((size_t)ka * n), dim3(256), 0, st, cur, prev, ep.alpha, ep.beta, (size_t)ka * n);
            for (int i = 2; i <= piece; ++i) {
                const double s2 = 1.0 / (2.0 / s0 - s1);
                DgEpilogue e2;
                e2.alpha = 2.0 * s2 / half;
                e2.c1 = cur;
                e2.ld1 = n;
                e2.beta = -2.0 * s2;
                e2.c2 = prev;
                e2.ld2 = n;
                e2.gamma = -s1 * s2;
                ok &= times_g(Gc, cur, prev, ka, n, st, w.scr, e2);      // the new term takes the place of the one before last
                std::swap(prev, cur);
                s1 = s2;
            }
            X = cur;
            tmp = prev;
            ok &= project_out(X, ka, n, Vr, l, w, st);
            ok &= orthonormalize(X, tmp, ka, n, last ? 2 : 1, w, st);
        }
    }
    return SVDP_OK;
}
