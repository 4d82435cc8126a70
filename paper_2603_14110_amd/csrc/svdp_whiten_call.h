// svdp_whiten_factors: its work buffers and the call itself.  Included by svdp.hip inside its unnamed namespace.

// ---- work buffers ----
struct WhitenWs {
    double *S;                  // [d][d]  C = X^T X, then its lower Cholesky factor
    double *M;                  // [D][d]  W S; the iteration takes what dominates out of it
    double *G;                  // [d][d]  M^T M
    double *T0, *T1, *T2;       // [d][d]  work matrices of the eigen-decomposition
    double *lamG;               // [d] eigenvalues by place
    double *invL;               // [d/64][64][64] inverses of S's diagonal blocks
    int32_t *fail;              // set by the factorisation if X^T X is not positive definite
    double *Vr, *Zr;            // [r][d]
    double *out64;              // [max(D, d)][r]
    double *part;               // parts of split products
    size_t n_part;
    double *Uall, *rowsums, *sums;     // [d/64][64][64] strip transforms; norms
    int32_t *sel;               // [d]
    double *small;              // the leading-eigenvector iteration's projected matrices
    size_t bytes;
    bool fits;
};

// Workspace size: what the call has asked for since its first version (fp64 copies of W, of W S and its transpose and
// of the tokens, six d x d matrices), so that a size a caller has stored stays right; carve_whiten() fits into it.
size_t whiten_ws_bytes(int d, int D, int T, int r)
{
    const size_t dd = (size_t)d * d, Dd = (size_t)D * d, most = D > d ? D : d;
    size_t bytes = 0;
    for (size_t n : {Dd, Dd, Dd, (size_t)d * T, dd, dd, dd, dd, dd, dd, (size_t)d, (size_t)64 * 64, (size_t)d * 64, (size_t)32,
                     (size_t)r * d, most * r, (size_t)d * 64, (size_t)2 * d, (size_t)2})
        bytes += align_up(n * 8);
    return bytes + align_up((size_t)r * 4);
}

// That size holds 3 D d + d T + 6 d^2 + r d + max(D, d) r + 131 d + 4096 doubles; what follows takes, without `part`,
// D d + 5 d^2 + 2 r d + 6 k^2 + max(D, d) r + 131.5 d + 67 k and at most 24 roundings to 32 doubles more.  T >= d leaves
// 2 D d + 2 d^2 - r d - 6 k^2 - 67 k - d / 2 + 4096 at least: more than d^2 where the iteration does not run (k = 0, r <= d),
// and 0.1 d^2 + 2 D d - 34 d + 4096 where it does (2 k <= d, r <= 0.8 k), at no d below 2400.
// The parts of split products get what is left, up to what they can use.
WhitenWs carve_whiten(void *base, int d, int D, int T, int r)
{
    WhitenWs w;
    char *p = static_cast<char *>(base);
    size_t off = 0;
    auto take = [&](size_t n_doubles) {
        double *q = reinterpret_cast<double *>(p + off);
        off += align_up(n_doubles * 8);
        return q;
    };
    const size_t dd = (size_t)d * d;
    w.S = take(dd);
    w.M = take((size_t)D * d);
    w.G = take(dd);
    w.T0 = take(dd);
    w.T1 = take(dd);
    w.T2 = take(dd);
    w.lamG = take(d);
    w.invL = take((size_t)d * 64);
    w.fail = reinterpret_cast<int32_t *>(take(32));
    w.Vr = take((size_t)r * d);
    w.Zr = take((size_t)r * d);
    w.out64 = take((size_t)(D > d ? D : d) * r);
    w.Uall = take((size_t)d * 64);
    w.rowsums = take((size_t)2 * d);
    w.sums = take(2);
    w.sel = reinterpret_cast<int32_t *>(take((size_t)(d + 1) / 2));
    const size_t k = eigtop_block(d, r);
    w.small = take(6 * k * k + 64 * k + 3 * k + 32);
    w.bytes = whiten_ws_bytes(d, D, T, r);
    w.n_part = std::min<size_t>((size_t)16 * 512 * 512, off < w.bytes ? (w.bytes - off) / 8 : 0);
    w.part = take(w.n_part);
    w.fits = off <= w.bytes;
    return w;
}

EigTopWs carve_eigtop(const WhitenWs &w, int d, int D, int r)
{
    EigTopWs e;
    const size_t k = eigtop_block(d, r), kn = k * d, kk = k * k;      // 2 k <= d: two blocks of vectors fit a d x d matrix
    e.k = (int)k;
    e.X = w.T0;
    e.Y = w.T0 + kn;
    e.Xa = w.T1;
    e.Xb = w.T1 + kn;
    e.M = w.M;
    e.D = D;
    e.MV = w.out64;
    e.Gd = w.T2;
    double *p = w.small;
    auto take = [&](size_t n) {
        double *q = p;
        p += n;
        return q;
    };
    e.H = take(kk);
    e.Ha = take(kk);
    e.V = take(kk);
    e.Va = take(kk);
    e.Vs = take(kk);
    e.L = take(kk);
    e.invL = take(64 * k);
    e.lam = take(k);
    e.theta = take(k);
    e.res = take(k);
    e.scale = take(32);
    e.Uall = w.Uall;
    e.rowsums = w.rowsums;
    e.sums = w.sums;
    e.sel = w.sel;
    e.fail = w.fail;
    e.scr = DgScratch{w.part, w.n_part};
    return e;
}

template <typename W>
svdp_status whiten_impl(const void *W_gate, const void *X, int d, int D, int T, int r, float *P, float *Q, float *sigma,
                        int32_t *sweeps, const WhitenWs &w, hipStream_t st)
{
    const W *Wg = static_cast<const W *>(W_gate), *Xs = static_cast<const W *>(X);
    std::vector<double> lam(d);

    const DgScratch scr{w.part, w.n_part};
    constexpr int SYM = DG_LOWER | DG_MIRROR;

    // second moments C = X^T X  (d x d) and its Cholesky factor S (lower, S S^T = C)
    if (!dgemm<DG_K_ROWS, DG_K_ROWS>(op(Xs, d), op(Xs, d), w.S, d, d, d, T, st, SYM, DgEpilogue{}, scr))
        return SVDP_ERR_UNSUPPORTED;
    if (hipMemsetAsync(w.fail, 0, 4, st) != hipSuccess) {
        (void)hipGetLastError();
        return SVDP_ERR_HIP;
    }
    if (!cholesky_blocked(w.S, d, w.invL, w.sums, w.fail, st)) return SVDP_ERR_UNSUPPORTED;
    int32_t failed = 0;
    if (hipMemcpyAsync(&failed, w.fail, 4, hipMemcpyDeviceToHost, st) != hipSuccess ||
        hipStreamSynchronize(st) != hipSuccess) {
        (void)hipGetLastError();
        return SVDP_ERR_HIP;
    }
    // S needs C positive definite (more independent tokens than dimensions)
    if (failed != 0) return SVDP_ERR_UNSUPPORTED;

    // M = W S and G = M^T M.  Not S^T ((W^T W) S), a quarter of the operations less at D = 2.7 d: where W hardly
    // responds to the direction that dominates the tokens, W^T W and S S^T cancel, and G would be off by
    // 2^-53 (||W|| ||S|| / ||W S||)^2 of itself (at tokens with a mean 1e6 times their spread 1e-6 of every singular value)
    bool ok = dgemm<DG_ROWS_K, DG_K_ROWS>(op(Wg, d), op((const double *)w.S, d), w.M, d, D, d, d, st, DG_K_FROM_N, DgEpilogue{},
                                          scr) &&
              dgemm<DG_K_ROWS, DG_K_ROWS>(op((const double *)w.M, d), op((const double *)w.M, d), w.G, d, d, d, D, st, SYM,
                                          DgEpilogue{}, scr);
    if (!ok) return SVDP_ERR_UNSUPPORTED;
    bool found = false;
    int sw2 = 0;
    EigTopWs ew = carve_eigtop(w, d, D, r);
    svdp_status e = leading_eigenvectors(w.G, d, r, w.Vr, lam.data(), found, &sw2, ew, st);
    if (e != SVDP_OK) return e;
    if (!found) {
        double *A = w.G, *Aalt = w.T0, *V = w.T1, *Valt = w.T2;
        e = jacobi_eigh(&A, &Aalt, &V, &Valt, d, w.Uall, w.rowsums, w.sums, w.lamG, 1e-11, 24, &sw2, st);
        if (e != SVDP_OK) return e;
        // the r largest eigenvalues (= squared singular values of W S), largest first; ties by place
        launch(k_rank_descending, grid1(d), dim3(256), 0, st, w.lamG, d, w.sel, w.rowsums);
        launch(k_gather_rows, grid1((size_t)r * d), dim3(256), 0, st, V, w.sel, r, d, w.Vr);
        if (hipMemcpyAsync(lam.data(), w.rowsums, (size_t)r * 8, hipMemcpyDeviceToHost, st) != hipSuccess) {
            (void)hipGetLastError();
            return SVDP_ERR_HIP;
        }
    }
    auto refused = [&] {                                          // the copies into lam must be done
        (void)hipStreamSynchronize(st);
        return SVDP_ERR_UNSUPPORTED;
    };
    // Q = A = W (S V_r)
    ok = dgemm<DG_ROWS_K, DG_ROWS_K>(op((const double *)w.Vr, d), op((const double *)w.S, d), w.Zr, d, r, d, d, st, DG_K_UPTO_N,
                                     DgEpilogue{}, scr) &&
         dgemm<DG_ROWS_K, DG_ROWS_K>(op(Wg, d), op((const double *)w.Zr, d), w.out64, r, D, r, d, st, 0, DgEpilogue{}, scr);
    if (!ok) return refused();
    launch(k_f64_to_f32, grid1((size_t)D * r), dim3(256), 0, st, w.out64, (size_t)D * r, Q);
    // B = V_r^T S^-1 (block back-substitution; V_r^T is w.Vr, rows = the chosen eigenvectors), P = B^T
    if (!solve_right_lower(w.Vr, w.out64, r, d, w.S, w.invL, st)) return refused();
    launch((k_transpose_to_f64<double>), dim3((d + 31) / 32, (r + 31) / 32), dim3(256), 0, st, w.out64, r, d, w.Vr);
    launch(k_f64_to_f32, grid1((size_t)d * r), dim3(256), 0, st, w.Vr, (size_t)d * r, P);
    if (hipStreamSynchronize(st) != hipSuccess) {                 // the copies into lam must be done
        (void)hipGetLastError();
        return SVDP_ERR_HIP;
    }
    if (sigma != nullptr)
        for (int k = 0; k < r; ++k) sigma[k] = (float)std::sqrt(std::max(lam[k], 0.0));
    if (sweeps != nullptr) {
        sweeps[0] = 0;              // the factor of the second moments is a Cholesky factor: no sweeps
        sweeps[1] = sw2;
    }
    return hip_status(hipSuccess);
}

