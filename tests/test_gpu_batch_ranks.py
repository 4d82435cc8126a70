"""Batches on the matrix cores at the sizes between the plain ones: scores of every rank and storage type, and rows of whole
128-byte lines that are no multiple of 512 elements, against the CPU oracle."""
import numpy as np
import pytest

import parity

pytestmark = pytest.mark.gpu

# d, D, r, B, storage; ranks around a column block (32 bf16 / 16 fp32 columns) and around the blocks held in registers (16)
RANKS = [(256, 64, 4, 3, "f32"), (264, 448, 12, 8, "f32"), (512, 320, 16, 5, "f32"), (300, 192, 20, 4, "f32"),
         (260, 640, 252, 8, "f32"), (128, 256, 260, 3, "f32"), (64, 128, 516, 6, "f32"),
         (256, 64, 8, 3, "bf16"), (264, 448, 40, 8, "bf16"), (1032, 320, 72, 5, "bf16"), (512, 192, 248, 4, "bf16"),
         (128, 256, 520, 8, "bf16"), (64, 128, 1032, 3, "bf16")]


def layer(torch, binding, d, D, r, B, dt, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    dtype = torch.float32 if dt == "f32" else torch.bfloat16
    mk = lambda *s: (torch.randn(*s, device="cuda", generator=g) / d ** 0.5).to(dtype)
    L = binding.DeviceLayer(mk(d, r), mk(D, r), torch.randn(D, device="cuda", generator=g) * 0.03, mk(D, d), mk(D, d), mk(D, d))
    return L, torch.randn(B, d, device="cuda", generator=g).to(dtype)


@pytest.mark.parametrize("d,D,r,B,dt", RANKS)
def test_scores_of_every_rank(d, D, r, B, dt):
    import torch
    from paper_2603_14110_amd import binding

    L, x = layer(torch, binding, d, D, r, B, dt, d + D + r)
    t = L.tensors
    ref = (x.double() @ t["P"].double()) @ t["Q"].double().T + t["b"].double()
    s = binding.predict(L, x)
    # two chains of d and of r fp32 additions: |error| <= (d + r) 2^-24 sum |terms|; far inside the bound used everywhere else
    assert float((s.double() - ref).abs().max()) <= 2e-5 * float(ref.abs().max())
    mask = torch.zeros(D // 64, dtype=torch.int64, device="cuda")
    binding.ffn_step(L, x, mask=mask)
    m2, _, _ = binding.compact(s)
    assert torch.equal(mask, m2)


@pytest.mark.parametrize("d,D,r,B,dt", [(256, 64, 8, 5, "bf16"), (64, 128, 40, 6, "bf16"), (128, 192, 544, 8, "bf16"),
                                         (128, 128, 64, 5, "bf16"), (64, 128, 20, 5, "f32")])
def test_scores_that_are_not_finite(d, D, r, B, dt):
    """An infinite or NaN t, a t between the largest bf16 and the largest fp32, and infinite or NaN rows of Q give both
    engines what the sum of the products is: the same infinities and NaN, everything else finite and right."""
    import torch
    from paper_2603_14110_amd import binding

    L, x = layer(torch, binding, d, D, r, B, dt, d + D + r)
    t = L.tensors
    P, Q = t["P"].abs(), t["Q"].clone()          # the sign of an infinite t is x's
    top = torch.finfo(torch.bfloat16).max
    P[0], P[1], P[2] = 2.0 ** -100, 0.0, 2.0 ** -120
    P[0, 0] = P[1, 0] = 1.0                      # column 0 of t: x[0] + x[1] + ...
    P[2, 3] = 4.0                                # column 3: overflows
    Q[0], Q[1] = Q[0].abs() + 0.25, -Q[1].abs() - 0.25
    Q[2, 0] = 1.0
    Q[5, 2], Q[6, 5], Q[7, 1] = torch.inf, -torch.inf, torch.nan
    Q[8] = 0.0
    x[1, 4] = torch.inf
    x[2, 0], x[2, 1], x[2, 2] = top, 1.5 * 2.0 ** 119, 0.0
    x[3, 2] = 2.0 ** 127
    x[4, 7] = torch.nan
    L = binding.DeviceLayer(P, Q, t["b"], t["W_gate"], t["W_up"], t["W_downT"])
    tt = (x.double().cpu() @ P.double().cpu()).float().double()
    assert tt[2, 0].isfinite() and tt[2, 0].to(torch.bfloat16).isinf() and tt[3, 3].isinf() and tt[3, 2].isfinite()
    terms = tt[:, None, :] * Q.double().cpu()[None]
    ref, size = terms.sum(-1) + t["b"].double().cpu(), terms.abs().sum(-1)
    ok = ref.isfinite()
    assert ref[1, 0] == torch.inf and ref[1, 1] == -torch.inf and ref[1, 8].isnan() and ref[2, 2].isfinite() and ok[0].sum() == D - 3
    for flags in (0, binding.FLAG_ENGINE_VECTOR, binding.FLAG_ENGINE_MATRIX):
        s = binding.predict(L.with_flags(flags), x)
        mask = torch.zeros(D // 64, dtype=torch.int64, device="cuda")
        binding.ffn_step(L.with_flags(flags), x, mask=mask)
        assert torch.equal(mask, binding.compact(s)[0]), flags
        s = s.cpu()
        assert torch.equal(s.isnan(), ref.isnan()), flags
        assert torch.equal(s[ref.isinf()].double(), ref[ref.isinf()]), flags
        # two chains of fp32 additions of d and r terms, as above, against the sum of the terms' sizes
        assert bool(((s.double() - ref).abs()[ok] <= 2e-5 * size[ok] + 1e-6).all()), flags


@pytest.mark.parametrize("d,D,B", [(64, 64, 8), (192, 640, 5), (576, 4160, 8), (1088, 2112, 3), (1856, 1152, 8)])
def test_rows_of_whole_lines(d, D, B):
    import torch
    import oracle
    from paper_2603_14110_amd import binding

    L, x = layer(torch, binding, d, D, 16, B, "bf16", d + D)
    f = {k: L.tensors[k].float().cpu().numpy() for k in ("W_gate", "W_up", "W_downT")}
    X = x.float().cpu().numpy()
    L = L.with_flags(binding.FLAG_ENGINE_MATRIX)
    idx = torch.zeros(D, dtype=torch.int32, device="cuda")
    nnz = torch.zeros(1, dtype=torch.int32, device="cuda")
    y = binding.ffn_step(L, x, idx=idx, nnz=nnz).cpu().numpy()
    lst = idx[: nnz.item()].cpu().numpy()
    parity.check_y(y, oracle.sparse_ffn(f["W_gate"], f["W_up"], f["W_downT"], X, lst), "bf16",
                   slack=parity.fp32_forward_bound(f, X, lst))
    yd = binding.dense_ffn(L, x).cpu().numpy()
    parity.check_y(yd, oracle.dense_ffn(f["W_gate"], f["W_up"], f["W_downT"], X), "bf16",
                   slack=parity.fp32_forward_bound(f, X, np.arange(D)))


@pytest.mark.parametrize("d,D,B", [(1032, 2112, 8), (1336, 1600, 5), (3128, 704, 8), (2104, 4224, 7), (8184, 320, 5)])
def test_rows_with_a_partial_line(d, D, B):
    """Layers of at least 2 M elements a matrix whose rows end inside a line: the default engine's rows, which are the matrix
    engine's (the same bits) and not the vector engine's (other sums)."""
    import torch
    import oracle
    from paper_2603_14110_amd import binding

    L, x = layer(torch, binding, d, D, 16, B, "bf16", d + D)
    f = {k: L.tensors[k].float().cpu().numpy() for k in ("W_gate", "W_up", "W_downT")}
    X = x.float().cpu().numpy()
    for drelu in (0, binding.FLAG_DRELU):
        idx = torch.zeros(D, dtype=torch.int32, device="cuda")
        nnz = torch.zeros(1, dtype=torch.int32, device="cuda")
        y = binding.ffn_step(L.with_flags(drelu), x, idx=idx, nnz=nnz)
        lst = idx.cpu().numpy()[: nnz.item()]
        parity.check_y(y.cpu().numpy(), oracle.sparse_ffn(f["W_gate"], f["W_up"], f["W_downT"], X, lst, drelu=bool(drelu)), "bf16",
                       slack=parity.fp32_forward_bound(f, X, lst))
        yd = binding.dense_ffn(L.with_flags(drelu), x)
        parity.check_y(yd.cpu().numpy(), oracle.sparse_ffn(f["W_gate"], f["W_up"], f["W_downT"], X, np.arange(D), drelu=bool(drelu)),
                       "bf16", slack=parity.fp32_forward_bound(f, X, np.arange(D)))
        for engine, same in ((binding.FLAG_ENGINE_MATRIX, True), (binding.FLAG_ENGINE_VECTOR, False)):
            assert torch.equal(binding.ffn_step(L.with_flags(drelu | engine), x), y) == same
            assert torch.equal(binding.dense_ffn(L.with_flags(drelu | engine), x), yd) == same


@pytest.mark.parametrize("d,D,dense,lists", [(512, 2560, True, False), (1024, 1088, True, False), (1024, 1024, False, False), (1000, 1088, True, False),
                                             (2048, 832, True, False), (2048, 768, False, False), (1024, 960, False, False),
                                             (4096, 512, True, True)])
def test_size_from_which_rows_are_on_the_matrix_cores(d, D, dense, lists):
    """The default engine at five and eight tokens, seen through bit patterns: over all rows above 1 M elements and 768 rows,
    over a list from 2 M elements on."""
    import torch
    import oracle
    from paper_2603_14110_amd import binding

    L, x = layer(torch, binding, d, D, 16, 8, "bf16", d + D)
    f = {k: L.tensors[k].float().cpu().numpy() for k in ("W_gate", "W_up", "W_downT")}
    X = x.float().cpu().numpy()
    M, V = L.with_flags(binding.FLAG_ENGINE_MATRIX), L.with_flags(binding.FLAG_ENGINE_VECTOR)
    idx, nnz = torch.arange(D, dtype=torch.int32, device="cuda"), torch.tensor([D], dtype=torch.int32, device="cuda")
    for B in (5, 8):
        ref = oracle.dense_ffn(f["W_gate"], f["W_up"], f["W_downT"], X[:B])
        slack = parity.fp32_forward_bound(f, X[:B], np.arange(D))
        for call, matrix in ((lambda l: binding.dense_ffn(l, x[:B]), dense), (lambda l: binding.sparse_ffn(l, x[:B], idx, nnz), lists)):
            y, ym, yv = call(L), call(M), call(V)
            assert not torch.equal(ym, yv) and torch.equal(y, ym if matrix else yv)
            parity.check_y(y.cpu().numpy(), ref, "bf16", slack=slack)


@pytest.mark.parametrize("d,D", [(8, 64), (56, 320), (120, 4160), (1032, 2112), (2104, 1088)])
def test_lists_with_a_partial_line(d, D):
    """Lists of the caller's own on the matrix cores, every batch size, rows that end inside a line: empty, one row, short and
    long, unsorted, with repeated entries and with entries outside the layer (which contribute nothing)."""
    import torch
    import oracle
    from paper_2603_14110_amd import binding

    L, x = layer(torch, binding, d, D, 8, 8, "bf16", d + D)
    f = {k: L.tensors[k].float().cpu().numpy() for k in ("W_gate", "W_up", "W_downT")}
    X = x.float().cpu().numpy()
    rng = np.random.default_rng(D)
    bad = rng.permutation(D)[: D // 2].astype(np.int32)
    bad[::5] = np.array([-1, D, D + 7, np.iinfo(np.int32).min, np.iinfo(np.int32).max], np.int32)[np.arange(bad[::5].size) % 5]
    lists = [np.zeros(0, np.int32), np.array([D - 1], np.int32), np.arange(D, dtype=np.int32), np.arange(0, D, 7, dtype=np.int32),
             rng.permutation(D).astype(np.int32), rng.integers(0, D, D).astype(np.int32), bad]
    for B, drelu in ((1, 0), (2, 0), (3, binding.FLAG_DRELU), (4, 0), (5, binding.FLAG_DRELU), (8, 0)):
        same = []
        for lst in lists:
            idx = torch.zeros(D, dtype=torch.int32, device="cuda")
            idx[: lst.size] = torch.from_numpy(lst).cuda()
            nnz = torch.tensor([lst.size], dtype=torch.int32, device="cuda")
            y = binding.sparse_ffn(L.with_flags(drelu | binding.FLAG_ENGINE_MATRIX), x[:B], idx, nnz)
            kept = lst[(lst >= 0) & (lst < D)]
            parity.check_y(y.cpu().numpy(), oracle.sparse_ffn(f["W_gate"], f["W_up"], f["W_downT"], X[:B], kept, drelu=bool(drelu)),
                           "bf16", slack=parity.fp32_forward_bound(f, X[:B], kept))
            assert kept.size > 0 or not y.any()
            same.append(torch.equal(y, binding.sparse_ffn(L.with_flags(drelu | binding.FLAG_ENGINE_VECTOR), x[:B], idx, nnz)))
        assert d < 64 or not all(same)                          # other sums than the vector engine's


@pytest.mark.parametrize("d,D,r,B,dt", [(4096, 128, 128, 8, "bf16"), (4104, 64, 136, 5, "bf16"), (264, 64, 256, 8, "bf16"), (8200, 64, 264, 8, "bf16"),
                                         (4352, 64, 512, 3, "bf16"), (512, 64, 520, 4, "bf16"), (4100, 64, 64, 8, "f32"), (256, 64, 68, 3, "f32"),
                                         (128, 64, 132, 8, "f32"), (64, 64, 260, 4, "f32"),
                                         (1024, 64, 384, 8, "bf16"), (1032, 64, 392, 4, "bf16"), (2048, 64, 192, 5, "f32"), (2052, 64, 196, 8, "f32"),
                                         (6144, 64, 96, 8, "bf16"), (6152, 64, 352, 3, "bf16"), (16384, 64, 128, 4, "bf16")])
def test_scores_at_the_edges_of_what_a_wave_holds(d, D, r, B, dt):
    """Ranks on both sides of 4, 8, 12 and 16 column blocks held at once; 1 to 64 partials of t, on both sides of the 4, 8 and 16
    requested at once; more and fewer slots of t than threads.  The bound of test_scores_of_every_rank."""
    test_scores_of_every_rank(d, D, r, B, dt)


@pytest.mark.parametrize("d,dt", [(10168, "bf16"), (5084, "f32")])
def test_rows_that_take_a_compute_units_whole_lds(d, dt):
    """Eight tokens and 32 rows a block: 8 d values and 9 x 32 words are 160 KB to the byte."""
    import torch
    from paper_2603_14110_amd import binding

    D, B, n = 8192, 8, 1000
    L, x = layer(torch, binding, d, D, 16, B, dt, d)
    assert 8 * d * L.tensors["W_gate"].element_size() + 9 * 4 * (D // 256) == 160 * 1024
    idx = torch.arange(0, D, device="cuda", dtype=torch.int32)
    idx[:n] = idx[5::8][:n].clone()
    y = binding.sparse_ffn(L, x, idx, torch.tensor([n], dtype=torch.int32, device="cuda"))
    rows = idx[:n].long()
    Wg, Wu, Wd = (L.tensors[k][rows].double() for k in ("W_gate", "W_up", "W_downT"))
    ref = ((x.double() @ Wg.T).clamp(min=0) * (x.double() @ Wu.T)) @ Wd
    # chains of d and of n fp32 additions, as for the scores above
    assert float((y.double() - ref).abs().max()) <= 2e-5 * float(ref.abs().max())


# B d values, and B + 1 words a row of a block's share (sequential: 2 B + 3), are 160 KB to the byte
@pytest.mark.parametrize("flag,B,d,D,dt", [("", 8, 10168, 8192, "bf16"), ("", 3, 10220, 4096, "f32"), ("sequential", 8, 10088, 8192, "bf16"),
                                             ("sequential", 8, 5044, 8192, "f32"), ("sequential", 3, 10196, 4096, "f32")])
def test_whole_lds_and_every_row(flag, B, d, D, dt):
    import torch
    from paper_2603_14110_amd import binding

    nb, es = 8 if B > 4 else 4, 4 if dt == "f32" else 2
    assert nb * d * es + (2 * nb + 3 if flag else nb + 1) * (D // 256) * 4 == 160 * 1024
    L, x = layer(torch, binding, d, D, 16, B, dt, d)
    dev = L.with_flags(binding.FLAG_REVALIDATE if flag else binding.FLAG_ENGINE_VECTOR)
    t = L.tensors
    g, u = x.double() @ t["W_gate"].double().T, x.double() @ t["W_up"].double().T
    h = g.clamp(min=0) * u
    idx = torch.arange(D, device="cuda", dtype=torch.int32)
    y = binding.sparse_ffn(dev, x, idx, torch.tensor([D], dtype=torch.int32, device="cuda"))
    mask = torch.zeros(D // 64, dtype=torch.int64, device="cuda")
    kept, nnz = torch.zeros(D, dtype=torch.int32, device="cuda"), torch.zeros(1, dtype=torch.int32, device="cuda")
    y2 = binding.ffn_step(dev, x, mask=mask, idx=kept, nnz=nnz)
    rows = kept[:int(nnz)].long()
    assert 0 < rows.numel() < D
    for out, ref in ((y, h @ t["W_downT"].double()), (y2, h[:, rows] @ t["W_downT"][rows].double()), (binding.dense_ffn(dev, x), h @ t["W_downT"].double())):
        # chains of d and of D fp32 additions, as for the scores above
        assert float((out.double() - ref).abs().max()) <= 2e-5 * float(ref.abs().max())


@pytest.mark.parametrize("d,D,r,B,dt", [(5120, 128, 512, 1, "bf16"), (4096, 128, 512, 2, "bf16"), (4104, 64, 520, 2, "bf16"), (5124, 64, 512, 1, "f32"),
                                         (16384, 64, 1024, 2, "bf16"), (2048, 64, 2048, 1, "f32")])
def test_scores_with_partials_left_for_a_loop(d, D, r, B, dt):
    """One and two tokens, more partials of t than the threads of a column request at the start; more columns than threads."""
    test_scores_of_every_rank(d, D, r, B, dt)


# 3 n d values on both sides of 64 MB (one and two tokens) and of 100 MB (more of them), where rows are requested with another cache hint
@pytest.mark.parametrize("d,dt,B,n", [(2048, "f32", 1, 2604), (2048, "f32", 2, 2605), (2052, "f32", 1, 2600), (2048, "f32", 3, 4069), (2048, "f32", 8, 4070),
                                       (4096, "bf16", 3, 4070), (4096, "bf16", 8, 4069), (4096, "bf16", 8, 4070), (4104, "bf16", 5, 4062)])
def test_long_lists(d, dt, B, n):
    import torch
    from paper_2603_14110_amd import binding

    es = 4 if dt == "f32" else 2
    limit = 64e6 if B <= 2 else 100e6
    assert abs(3 * n * d * es - limit) <= 0.002 * limit
    L, x = layer(torch, binding, d, (n + 127) // 64 * 64, 16, B, dt, n)
    D = L.tensors["W_gate"].shape[0]
    idx = torch.randperm(D, device="cuda", generator=torch.Generator(device="cuda").manual_seed(n)).to(torch.int32)
    y = binding.sparse_ffn(L, x, idx, torch.tensor([n], dtype=torch.int32, device="cuda"))
    rows = idx[:n].long()
    Wg, Wu, Wd = (L.tensors[k][rows].double() for k in ("W_gate", "W_up", "W_downT"))
    ref = ((x.double() @ Wg.T).clamp(min=0) * (x.double() @ Wu.T)) @ Wd
    # chains of d and of n fp32 additions, as for the scores above
    assert float((y.double() - ref).abs().max()) <= 2e-5 * float(ref.abs().max())
