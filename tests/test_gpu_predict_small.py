"""The one-launch predictor of small layers (k_predict_small) against the two kernels it stands for, which
svdp_ffn_step_glued still runs: every sum has one order in both, so mask, list and y have the same bits.  The two kernels are
compared with the oracle in test_gpu_parity.py; the scores are compared with a 64-bit product here."""
import pytest

pytestmark = pytest.mark.gpu

SHAPES = [  # d, D, r, storage; P has 1 to 4 tiles of 256 x 32
    (256, 1024, 32, "f32"),
    (264, 448, 40, "f32"),        # ragged last tile both ways
    (1024, 320, 24, "f32"),       # four tiles of rows
    (64, 64, 4, "f32"),           # the smallest
    (200, 128, 128, "f32"),       # four tiles of columns, 32 lanes a row
    (256, 2048, 32, "bf16"),
    (520, 192, 8, "bf16"),        # three tiles of rows, the last of 8 rows
    (72, 640, 120, "bf16"),       # four tiles of columns, the last ragged
    (1000, 576, 16, "bf16"),
    (1032, 576, 16, "bf16"),      # five tiles: the two kernels themselves
]


@pytest.mark.parametrize("d,D,r,dt", SHAPES)
def test_one_launch_predictor_gives_the_two_kernels_bits(d, D, r, dt):
    import torch
    from paper_2603_14110_amd import binding

    g = torch.Generator(device="cuda")
    g.manual_seed(d + D)
    dtype = torch.float32 if dt == "f32" else torch.bfloat16
    mk = lambda *s: (torch.randn(*s, device="cuda", generator=g) / d ** 0.5).to(dtype)
    L = binding.DeviceLayer(mk(d, r), mk(D, r), torch.randn(D, device="cuda", generator=g) * 0.03, mk(D, d), mk(D, d), mk(D, d))
    new = lambda: (torch.zeros(D // 64, dtype=torch.int64, device="cuda"),
                   torch.full((D,), -1, dtype=torch.int32, device="cuda"), torch.zeros(1, dtype=torch.int32, device="cuda"))
    x, (mask, idx, nnz) = torch.empty(1, d, dtype=dtype, device="cuda"), new()
    y = binding.ffn_step_glued(L, mk(1, d), torch.randn(1, d, device="cuda", generator=g), torch.zeros(d, device="cuda"), x,
                               mask=mask, idx=idx, nnz=nnz)
    m2, i2, n2 = new()
    y2 = binding.ffn_step(L, x, mask=m2, idx=i2, nnz=n2)
    assert torch.equal(mask, m2) and torch.equal(idx, i2) and torch.equal(nnz, n2) and torch.equal(y, y2)
    s = binding.predict(L, x)
    ref = (x.double() @ L.tensors["P"].double()) @ L.tensors["Q"].double().T + L.tensors["b"].double()
    assert float((s.double() - ref).abs().max()) <= 2e-5 * float(ref.abs().max())
    m3, i3, n3 = binding.compact(s)
    assert torch.equal(m2, m3) and torch.equal(n2, n3)
