"""Workloads of the sparse FFN library, as a user's program drives it.

A case is a dict of plain values; its ``kind`` says which public entry points one pass goes through:

  step    binding.ffn_step: one layer, one batch of decode tokens (predictor, mask, list, sparse FFN), launched eagerly
  stack   stack.FFNStack.step: one decode step through several layers, captured once as a HIP graph and replayed
  list    binding.sparse_ffn: the FFN over an index list the caller brings
  dense   binding.dense_ffn: every neuron (layers that are not sparse enough, and the baseline)
  scores  binding.predict + binding.compact: a caller that looks at the scores before it makes the list
  stats   binding.calib_stats: damage weights and proxy scores of a calibration set
  bias    binding.calib_bias: greedy thresholds from such statistics
  whiten  binding.whiten_factors: predictor factors from the gate matrix and calibration tokens

Layers and tokens are made on the GPU with the distributions of ``paper_2603_14110_amd.synth``: a gate matrix of
low rank plus noise, shifted along the tokens' mean direction so that about 90 % of the gate products are negative,
unit-variance up and down projections, and a bias that keeps the neurons which calibration tokens activate.
"""
from __future__ import annotations

import torch

from paper_2603_14110_amd import binding
from paper_2603_14110_amd.stack import FFNStack

FLAGS = {"": 0, "drelu": binding.FLAG_DRELU, "revalidate": binding.FLAG_REVALIDATE}
DTYPES = {"bf16": torch.bfloat16, "f32": torch.float32}
K_DOM = 64           # dominant rank of a generated gate matrix
CAL_TOKENS = 512     # tokens that set a generated layer's shift and bias


def listed():
    return [
        # the smallest layer in use (a test-sized fp32 model): nothing but launches and latency
        dict(name="step tiny f32", kind="step", d=256, D=1024, r=32, B=1, dtype="f32", flags="", sparsity=0.90),
        # the ordinary call: one token through one 7B-shaped layer, mask and list wanted by the caller
        dict(name="step 7b", kind="step", d=4096, D=11008, r=256, B=1, dtype="bf16", flags="", sparsity=0.90),
        # a whole decode step of a model: layers of different sparsity, one graph per token, weights from HBM
        dict(name="stack 7b x8 graph", kind="stack", d=4096, D=11008, r=256, layers=8, dtype="bf16", lo=0.80, hi=0.95),
        # a cheap low-rank predictor that over-predicts, corrected by the gate (sequential pipeline)
        dict(name="step 7b r32 sequential", kind="step", d=4096, D=11008, r=32, B=1, dtype="bf16", flags="revalidate",
             sparsity=0.90),
        # a few sequences decoded together: wide layer, high predictor rank
        dict(name="step qwen b4", kind="step", d=3584, D=18944, r=512, B=4, dtype="bf16", flags="", sparsity=0.90),
        # the largest decode batch: the union of eight masks is half dense
        dict(name="step mistral b8", kind="step", d=4096, D=14336, r=256, B=8, dtype="bf16", flags="", sparsity=0.90),
        # ragged sizes, both branches rectified, a list of the caller's own
        dict(name="list ragged b2", kind="list", d=2824, D=7552, r=200, B=2, dtype="bf16", flags="drelu", n=1507),
        # the largest dense layer
        dict(name="dense 13b", kind="dense", d=5120, D=13824, r=320, B=1, dtype="bf16", flags=""),
        # offline: statistics of a calibration set (the two wide contractions of the bias calibration)
        dict(name="stats 7b", kind="stats", d=4096, D=11008, r=256, T=2048),
        # offline: the greedy thresholds themselves
        dict(name="bias 7b", kind="bias", D=11008, T=2048, eta=16, level=0.90),
        # offline: data-aware factors, of a small and of a 7B-shaped gate matrix
        dict(name="whiten small", kind="whiten", d=1024, D=2752, T=2048, r=64, dtype="bf16"),
        dict(name="whiten 7b", kind="whiten", d=4096, D=11008, T=8192, r=256, dtype="bf16"),
    ]


def _log(rng, lo, hi):
    return lo * (hi / lo) ** rng.random()


def _mult(v, m, lo):
    return max(lo, int(round(v / m)) * m)


def draw(rng):
    """One more case: any kind, sizes over the whole range of the listed ones (about half of them on no round number)."""
    kind = rng.choice(["step"] * 5 + ["stack", "list", "list", "dense", "scores", "stats", "bias", "whiten"])
    dtype = rng.choice(["bf16", "bf16", "bf16", "f32"])
    if kind in ("stats", "whiten", "stack"):
        dtype = rng.choice(["bf16", "bf16", "f32"]) if kind == "whiten" else "bf16"
    unit = rng.choice([8, 8, 64, 128, 512])
    d = _mult(_log(rng, 256, 5120 if dtype == "bf16" else 2048), unit, 256)
    D = _mult(min(d * rng.uniform(2.5, 5.3), 18944), 64, 512)
    r = _mult(_log(rng, 16, min(512, d / 2)), rng.choice([8, 16, 32]), 16)
    B = rng.choice([1, 1, 1, 2, 3, 4, 5, 6, 8])
    if kind == "step":
        return dict(kind=kind, d=d, D=D, r=r, B=B, dtype=dtype, flags=rng.choice(["", "", "", "drelu", "revalidate"]),
                    sparsity=round(rng.uniform(0.80, 0.95), 3))
    if kind == "stack":
        return dict(kind=kind, d=d, D=min(D, 13824), r=r, layers=rng.randint(2, 6), dtype=dtype, lo=0.80, hi=0.95)
    if kind == "list":
        return dict(kind=kind, d=d, D=D, r=r, B=B, dtype=dtype, flags=rng.choice(["", "drelu", "revalidate"]),
                    n=int(_log(rng, 1, D)))
    if kind == "dense":
        return dict(kind=kind, d=d, D=D, r=r, B=B, dtype=dtype, flags=rng.choice(["", "drelu"]))
    if kind == "scores":
        return dict(kind=kind, d=d, D=D, r=r, B=B, dtype=dtype, flags="", sparsity=round(rng.uniform(0.80, 0.95), 3))
    if kind == "stats":
        return dict(kind=kind, d=d, D=D, r=r, T=int(_log(rng, 100, 4096)))
    if kind == "bias":
        return dict(kind=kind, D=D, T=int(_log(rng, 64, 4096)), eta=int(_log(rng, 1, 64)),
                    level=round(rng.uniform(0.6, 0.95), 3))
    d = _mult(_log(rng, 256, 2560), 64, 256)
    return dict(kind=kind, d=d, D=_mult(d * rng.uniform(2.5, 4.0), 64, 512), T=int(d * rng.uniform(1.2, 3.0)),
                r=_mult(_log(rng, 16, d / 4), 8, 16), dtype=dtype)


# ---- inputs ---------------------------------------------------------------------------------------------------------

def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _normal(g, *shape):
    return torch.randn(*shape, device="cuda", generator=g)


def _tokens(g, u, n, dtype):
    """n tokens x = 2u + N(0, 1)^d in the storage type."""
    return (2.0 * u[None, :] + _normal(g, n, u.numel())).to(dtype)


def _projection(g, D, d, dtype):
    return _normal(g, D, d).mul_(d ** -0.5).to(dtype)


def _gate(g, u, D, d, sparsity, dtype):
    """W_gate = 0.8 A B^T + 0.2 noise - alpha 1 u^T in the storage type, B, and calibration tokens; alpha puts
    the wanted share of the gate products below zero."""
    k = min(K_DOM, d // 16)
    A, Bm = _normal(g, D, k).mul_(k ** -0.25), _normal(g, d, k).mul_(k ** -0.25)
    W = (A @ Bm.T).mul_(0.8).add_(_normal(g, D, d).mul_(0.2 * d ** -0.5))
    X = _tokens(g, u, CAL_TOKENS, dtype)
    lift = (X[:64].float() @ W[:4096].T) / (X[:64].float() @ u)[:, None].clamp(min=0.25)
    alpha = torch.sort(lift.flatten())[0][int(sparsity * lift.numel())]
    return W.sub_(alpha * u[None, :]).to(dtype), Bm, X


def _factors(g, W, Bm, u, X, r, dtype):
    """Rank-r predictor in the storage type: the gate matrix projected onto r directions, its dominant ones first,
    and the bias that keeps every neuron a calibration token activates."""
    d = W.shape[1]
    P = torch.cat([u[:, None], Bm, _normal(g, d, r)], dim=1)[:, :r].double()
    P = P / P.norm(dim=0, keepdim=True)
    G = torch.linalg.inv((P.T @ P).cpu()).cuda()
    Q = (W.float() @ (P @ G).float())
    P, Q = P.to(dtype).contiguous(), Q.to(dtype).contiguous()
    S = (X.float() @ P.float()) @ Q.float().T
    on = (X.float() @ W.float().T) > 0
    tau = torch.where(on, S, torch.inf).amin(dim=0)
    tau = torch.where(on.any(dim=0), tau - 1e-5 * tau.abs(), S.amax(dim=0))
    return P, Q, -tau


def _layer(g, c, sparsity):
    d, D, r, dtype = c["d"], c["D"], c["r"], DTYPES[c["dtype"]]
    u = _normal(g, d)
    u = u / u.norm()
    W, Bm, X = _gate(g, u, D, d, sparsity, dtype)
    P, Q, b = _factors(g, W, Bm, u, X, r, dtype)
    return P, Q, b, W, u


def _random_layer(g, c):
    """Weights without structure, for the entry points that take no predictor."""
    d, D, r, dtype = c["d"], c["D"], c["r"], DTYPES[c["dtype"]]
    return binding.DeviceLayer(_projection(g, d, r, dtype), _projection(g, D, r, dtype), torch.zeros(D, device="cuda"),
                               _projection(g, D, d, dtype), _projection(g, D, d, dtype), _projection(g, D, d, dtype),
                               flags=FLAGS[c["flags"]])


def _typical_batch(g, u, P, Q, b, B, dtype):
    """Of 48 batches the one whose list length is nearest their mean (a token's own density varies from 0 to 80 %),
    and the bias moved off its scores wherever one is within rounding of zero, so that the mask has one right value."""
    X = _tokens(g, u, 48 * B, dtype)
    n = ((X.float() @ P.float()) @ Q.float().T + b > 0).view(48, B, -1).any(dim=1).sum(dim=1).float()
    k = int((n - n.mean()).abs().argmin())
    x = X.view(48, B, -1)[k].contiguous()
    s0 = (x.double() @ P.double()) @ Q.double().T
    for _ in range(4):
        s = s0 + b.double()
        top = s.abs().amax()
        close = (s.abs() < 2e-5 * top).any(dim=0)
        b = torch.where(close, b - 1e-4 * top.float(), b)
    return x, b.contiguous()


def prepare(case, seed):
    c, g = case, _gen(seed)
    kind = c["kind"]
    if kind == "stack":
        dtype = DTYPES[c["dtype"]]
        layers, us = [], []
        for l in range(c["layers"]):
            share = l / max(1, c["layers"] - 1)
            P, Q, b, W, u = _layer(g, c, c["lo"] + (c["hi"] - c["lo"]) * share)
            up, down = (_projection(g, c["D"], c["d"], dtype) for _ in range(2))
            layers.append(binding.DeviceLayer(P, Q, b, W, up, down))
            us.append(u)
        shifts = [2.0 * u for u in us[1:]] + [torch.zeros_like(us[0])]
        st, x0 = FFNStack(layers, shifts), _tokens(g, us[0], 1, dtype)[0]
        st.step(x0)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            out = st.step(x0)
        return dict(kind=kind, stack=st, graph=graph, x0=x0, out=out)
    if kind in ("step", "scores"):
        dtype, B = DTYPES[c["dtype"]], c["B"]
        P, Q, b, W, u = _layer(g, c, c["sparsity"])
        x, b = _typical_batch(g, u, P, Q, b, B, dtype)
        up, down = (_projection(g, c["D"], c["d"], dtype) for _ in range(2))
        L = binding.DeviceLayer(P, Q, b, W, up, down, flags=FLAGS[c["flags"]])
        return dict(kind=kind, layer=L, x=x, ws=L.workspace(B), y=torch.zeros(B, c["d"], device="cuda"),
                    mask=torch.zeros(c["D"] // 64, dtype=torch.int64, device="cuda"),
                    idx=torch.full((c["D"],), -1, dtype=torch.int32, device="cuda"),
                    nnz=torch.zeros(1, dtype=torch.int32, device="cuda"))
    if kind in ("list", "dense"):
        L = _random_layer(g, c)
        s = dict(kind=kind, layer=L, x=_normal(g, c["B"], c["d"]).to(L.dtype), ws=L.workspace(c["B"]),
                 y=torch.zeros(c["B"], c["d"], device="cuda"))
        if kind == "list":
            idx = torch.randperm(c["D"], device="cuda", generator=g)[:c["n"]].sort()[0].to(torch.int32)
            s["idx"] = torch.cat([idx, torch.full((c["D"] - c["n"],), -1, dtype=torch.int32, device="cuda")])
            s["nnz"] = torch.tensor([c["n"]], dtype=torch.int32, device="cuda")
        return s
    if kind == "stats":
        c = dict(c, dtype="bf16")
        P, Q, b, W, u = _layer(g, c, 0.90)
        up, down = (_projection(g, c["D"], c["d"], torch.bfloat16) for _ in range(2))
        return dict(kind=kind, layer=binding.DeviceLayer(P, Q, b, W, up, down), X=_tokens(g, u, c["T"], torch.bfloat16))
    if kind == "bias":
        # statistics with the structure of calib_stats' own: the score tracks the true gate up to noise, one gate
        # product in ten is positive, and the damage weight is zero where it is not
        z = _normal(g, c["D"], c["T"]) + _normal(g, c["D"], 1).mul_(0.5)
        gate = (z - 1.4).clamp_(min=0)
        w = (gate * _normal(g, c["D"], c["T"])).square_()
        s = z.add_(_normal(g, c["D"], c["T"]).mul_(0.3))
        return dict(kind=kind, w=w, s=s, eta=c["eta"], need=binding.calib_need(c["level"], c["D"], c["T"]))
    if kind == "whiten":
        d, dtype = c["d"], DTYPES[c["dtype"]]
        u = _normal(g, d)
        u = u / u.norm()
        W, _, _ = _gate(g, u, c["D"], d, 0.90, dtype)
        # correlated tokens: without them whitening would have nothing to do
        decay = torch.exp(torch.arange(d, device="cuda") * (-2.0 / d))[torch.randperm(d, device="cuda", generator=g)]
        X = ((2.0 * u[None, :] + _normal(g, c["T"], d)) * decay[None, :]).to(dtype)
        return dict(kind=kind, W=W, X=X, r=c["r"])
    raise ValueError(kind)


# ---- one pass -------------------------------------------------------------------------------------------------------

def run(state):
    s = state
    kind = s["kind"]
    if kind == "step":
        y = binding.ffn_step(s["layer"], s["x"], ws=s["ws"], out=s["y"], mask=s["mask"], idx=s["idx"], nnz=s["nnz"])
        return {"y": y, "mask": s["mask"], "idx": s["idx"], "nnz": s["nnz"]}
    if kind == "stack":
        s["graph"].replay()
        return {"x": s["out"], "y": s["stack"].y}
    if kind == "list":
        return binding.sparse_ffn(s["layer"], s["x"], s["idx"], s["nnz"], ws=s["ws"], out=s["y"])
    if kind == "dense":
        return binding.dense_ffn(s["layer"], s["x"], ws=s["ws"], out=s["y"])
    if kind == "scores":
        scores = binding.predict(s["layer"], s["x"], ws=s["ws"])
        mask, idx, nnz = binding.compact(scores)
        return {"scores": scores, "mask": mask, "idx": idx, "nnz": nnz}
    if kind == "stats":
        w, sc = binding.calib_stats(s["layer"], s["X"])
        return {"w": w, "s": sc}
    if kind == "bias":
        b, k, steps, _ = binding.calib_bias(s["w"], s["s"], s["eta"], s["need"])
        return {"b": b, "k": k, "steps": steps}
    # the columns of the two factors are unique only up to sign (and rotation where singular values meet): what a
    # program evaluates, and what is returned, is the predictor they make, W_gate ~ Q P^T, with the singular values
    P, Q, sigma, _ = binding.whiten_factors(s["W"], s["X"], s["r"])
    return {"gate": Q @ P.T, "sigma": sigma}


# ---- what a pass cannot do without ----------------------------------------------------------------------------------

def work(case):
    c, kind = case, case["kind"]
    w = 4 if c.get("dtype") == "f32" else 2
    d, D, r, B = c.get("d", 0), c["D"], c.get("r", 0), c.get("B", 1)
    pred = (d + D) * r * w + 4 * D
    io = B * d * w + 4 * B * d
    if kind in ("step", "stack"):
        # share of the neurons that B tokens activate together, of independent tokens at the case's sparsity
        share = 1.0 - (c["sparsity"] if kind == "step" else 0.5 * (c["lo"] + c["hi"])) ** B
        n = share * D
        L = c.get("layers", 1)
        return {"bytes": L * (pred + 3 * n * d * w + io), "flops": L * 2 * B * ((d + D) * r + 3 * n * d)}
    if kind in ("list", "dense"):
        n = c["n"] if kind == "list" else D
        return {"bytes": 3 * n * d * w + io, "flops": 6 * B * n * d}
    if kind == "scores":
        return {"bytes": pred + B * d * w + 4 * B * D, "flops": 2 * B * (d + D) * r}
    T = c["T"]
    if kind == "stats":
        return {"bytes": 3 * D * d * 2 + T * d * 2 + (d + D) * r * 2 + 8 * D * T,
                "flops": 4 * D * T * d + 2 * T * r * d + 2 * D * T * r}
    if kind == "bias":
        return {"bytes": 8 * D * T + 8 * D, "flops": 0}
    # second moments and Gram matrix by their lower halves, the product with a triangular factor, the reduction
    # of a d x d symmetric matrix and r of its eigenvectors, the two factor products (all in 64 bits)
    return {"bytes": (D + T) * d * w + 4 * (D + d) * r,
            "flops": d * d * T + 2 * D * d * d + 5 * d * d * d / 3 + 2 * D * d * r + 3 * d * d * r}


def tolerance(case):
    # each about four times the distance from the same path evaluated in 64 bits
    kind = case["kind"]
    if kind in ("step", "list", "dense", "scores"):
        # exact products of stored values, fp32 sums in any order (measured 1.4e-7 .. 5e-7, largest 2.2e-6);
        # the mask and the list are whole numbers and exact
        return {"rel": 2e-6, "max": 2e-5}
    if kind == "stack":
        return {"rel": 1e-2, "max": 0.2}             # bf16 tokens handed from layer to layer
    if kind == "stats":
        return {"rel": 4e-6, "max": 4e-5}            # measured 1.0e-6, largest 9.7e-6
    if kind == "bias":
        return "exact"
    return {"rel": 2e-6, "max": 2e-5}                # fp32 factors of a 64-bit decomposition, one fp32 product
