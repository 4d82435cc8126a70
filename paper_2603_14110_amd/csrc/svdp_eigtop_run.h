// The r leading eigenvectors of a symmetric positive semi-definite matrix G [n][n] without its other n - r: a block of
// k > r vectors is filtered by Chebyshev polynomials of G that are small on [0, b], b = the block's smallest Ritz value,
// and large above (subspace iteration with Rayleigh-Ritz).  Almost all of it is k x n x n products on the fp64 matrix
// cores, 4 to 35 of them; block Jacobi runs on the k x k projections only.  Included by svdp.hip after
// svdp_whiten_run.h's helpers, inside its unnamed namespace.
//
//   start    k pseudo-random rows, three times X <- orth(X G)
//   repeat   Rayleigh-Ritz: H = X G X^T, its eigenvectors rotate X; residuals of the wanted vectors; done if small
//            vectors that have settled leave the block: G <- G - v theta v^T, so that a few dominant directions
//            (the mean of the tokens carries 1e8 times the energy of the rest) do not limit the filter's degree
//            X <- orth(p(G) X), as many degrees as the Ritz values say are missing, in pieces of at most EIG_PIECE that
//            also keep X's condition number below EIG_AMPLIFY
//
// Accuracy: the residuals of the block's wanted vectors together end below 2e-13 of ||G||_F, those of the r that left it
// below 3e-14 sqrt(r); the Jacobi path stops at an off-diagonal norm of 1e-11 of it.
// Measured (bf16, whole call), full Jacobi -> this: d = 4096, r = 256: 401 -> 31 ms (33 products of 256 to 320 x 4096 x
// 4096 at 0.16 to 0.22 ms, two projections of 11 Jacobi sweeps together); d = 1024, r = 64: 43.6 -> 3.2 ms; d = 2560,
// r = 640: 183 -> 45 ms.  With b fixed between projections and pieces as long as the condition number allowed, the first
// took three projections and 50 ms: b starts at 0.65 of where it ends, which costs three quarters of the filter's rate.
// Where it does not apply (block of more than half the dimension; no gap in reach behind the wanted vectors; X loses
// rank, e.g. G of rank below r) the full Jacobi decomposition runs instead, on the untouched G.

constexpr double EIG_TOL = 2e-13;           // sqrt(sum of squared residuals of the wanted vectors) / ||G||_F
constexpr double EIG_TOL_JACOBI = 1e-13;    // of the projected problems (off-diagonal / total Frobenius norm)
constexpr double EIG_TOL_FIRST = 1e-12;     // of the first one, which only has to separate what dominates
constexpr double EIG_SETTLED = 3e-14;       // residual / ||G||_F of one vector that may leave the block
constexpr double EIG_AMPLIFY = 1e5;         // largest over smallest filter value between two orthogonalisations
constexpr double EIG_PIECE = 8.0;           // largest degree of a piece of the filter
constexpr double EIG_SHIFT = 4e-13;         // of the first Cholesky QR pass (above k_chol_diag's bound of 1e-13)

// Rows of the block for r wanted vectors: a quarter more (at least 32), so that the filter has a gap to work with, in
// whole Jacobi strips; 0 where the Jacobi decomposition of all of G is the better way: from n = 256 on the block wins on
// every spectrum tried (whole call 3.9 to 4.4 against 5.0 to 8.1 ms at r = 64), at n = 128 it loses on decaying ones (2.2
// against 1.6 ms).
inline int eigtop_block(int n, int r)
{
    const int k = round_up(r + std::max(32, r / 4), BJ_S);
    return n >= 256 && 2 * k <= n ? k : 0;
}

struct EigTopWs {
    int k;                              // eigtop_block(n, r)
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

// X <- X - (X Vl^T) Vl for the l rows of Vl and the ka of X.  The coefficients lie in Vs with the full block's stride: as
// vectors leave the block, l outgrows ka, but never w.k (l < r < w.k).  false: it would not fit, nothing was done.
bool project_out(double *X, int ka, int n, const double *Vl, int l, const EigTopWs &w, hipStream_t st)
{
    if (l == 0) return true;
    if (l > w.k || ka > w.k) return false;
    dgemm<DG_ROWS_K, DG_ROWS_K>(op((const double *)X, n), op(Vl, n), w.Vs, w.k, ka, l, n, st, 0, DgEpilogue{}, w.scr);
    dgemm<DG_ROWS_K, DG_K_ROWS>(op((const double *)w.Vs, w.k), op(Vl, n), X, n, ka, n, l, st, 0, minus_from(X, n));
    return true;
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
        orthonormalize(X, tmp, k, n, p < 2 ? 1 : 3, w, st);
    }
    const double *Gc = G;
    double norm = 0.0, last_err = 1e300;
    int l = 0, ka = k, products = 4, piece = 0;             // vectors that left the block; rows of the block
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
            jacobi_eigh(&A, &Aa, &V, &Va, ka, w.Uall, w.rowsums, w.sums, w.lam, cycle == 0 ? EIG_TOL_FIRST : EIG_TOL_JACOBI, 24, &sw, st);
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
        const double b = std::max(theta[ka - 1], 1e-15 * norm), margin = 10.0;
        // no gap in reach: the full decomposition would be done sooner
        const double apart = std::acosh(std::max(2.0 * theta[need - 1] / b - 1.0, 1.0));
        if (!(std::log(std::max(err / EIG_TOL, 2.0)) / apart * ka < 16.0 * n - (double)products * ka)) return SVDP_OK;
        // Settled vectors leave the block.  What is left of their residual couples them to the rest of G by as little, far
        // below the filter's edge, so it does not grow.
        int out = 0;
        while (out < need && std::sqrt(res[out]) < EIG_SETTLED * norm && theta[out] > 2.0 * theta[need - 1]) ++out;
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
                if (!project_out(X, ka, n, Vr, l, w, st)) return SVDP_OK;
                orthonormalize(X, tmp, ka, n, 1, w, st);
            }
        }
        // Filter, in pieces.  Before each but the first, b follows the smallest Rayleigh quotient of the block, which is
        // near its smallest Ritz value (the rows stay in the order of the Ritz values): it rises while the block's last rows
        // settle, and the rate hangs on it, because what lies outside the block is only damped as far as b reaches.
        double bound = b, todo = std::log(std::max(err / EIG_TOL * margin, 2.0));
        double wanted = theta[need - 1];
        auto growth = [](double value, double edge) { return std::acosh(std::max(2.0 * value / edge - 1.0, 1.0)); };
        int single = 0;
        for (bool first = true, last = false; !last; first = false) {
            double *prev = X, *cur = X == w.X ? w.Xa : w.X;
            if (!first) {
                times_g(Gc, X, cur, ka, n, st, w.scr);
                hipLaunchKernelGGL(k_rayleigh, dim3(ka), dim3(256), 0, st, X, cur, n, w.res);
                if (hipMemcpyAsync(res, w.res, (size_t)ka * 8, hipMemcpyDeviceToHost, st) != hipSuccess ||
                    hipStreamSynchronize(st) != hipSuccess)
                    return hip_failed();
                std::sort(res, res + ka, std::greater<double>());
                const double lowest = res[ka - 1];
                wanted = std::max(wanted, res[r - l - 1]);         // has risen, too
                if (!(lowest < wanted)) break;                     // (also NaN) the next projection tells more
                // what the last piece gained where the new bound now is
                todo += piece * growth(lowest, bound);
                bound = std::max(bound, lowest);
            }
            const double rate = growth(wanted, bound), left = std::ceil(todo / rate);
            if (!(left * ka < 16.0 * n - (double)products * ka)) return SVDP_OK;
            piece = (int)std::max(1.0, std::min({EIG_PIECE, std::floor(std::acosh(EIG_AMPLIFY) / std::max(growth(top, bound), 1e-3)), left}));
            last = piece >= left || (piece == 1 && ++single == 3);  // a dominant direction keeps the pieces short: project, it may have settled
            todo -= piece * rate;
            products += piece;
            const double half = 0.5 * bound, s0 = half / (top - half);
            double s1 = s0;
            DgEpilogue ep;
            ep.alpha = s1 / half;
            ep.c1 = prev;
            ep.ld1 = n;
            ep.beta = -s1;
            if (first) times_g(Gc, prev, cur, ka, n, st, w.scr, ep);
            else hipLaunchKernelGGL(k_combine, grid1((size_t)ka * n), dim3(256), 0, st, cur, prev, ep.alpha, ep.beta, (size_t)ka * n);
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
                times_g(Gc, cur, prev, ka, n, st, w.scr, e2);      // the new term takes the place of the one before last
                std::swap(prev, cur);
                s1 = s2;
            }
            X = cur;
            tmp = prev;
            if (!project_out(X, ka, n, Vr, l, w, st)) return SVDP_OK;
            orthonormalize(X, tmp, ka, n, last ? 2 : 1, w, st);
        }
        products += 1;
    }
    return SVDP_OK;
}
