"""The act' factors of ReLU stacks, stored as bits (MGRIT_ACT_VALUES=0), against the same factors stored as values (=1): every kernel
that writes or reads them, at widths and channel counts whose rows end inside a byte group of another row, at images whose last
block of pixels is short.  The arithmetic is the same, so states and gradients agree bit for bit, infinities (0 times one is
NaN) included."""
import numpy as np
import pytest

import mgrit_inputs as I
from tests.gpu_util import GpuProblem
from tests.test_gpu_mixed import GpuMixed

pytestmark = pytest.mark.gpu


def _dense(q, B, N, dtype, m=4, levels=2):
    return I.reduced(I.cfg5(1), name=f"bits_dense_q{q}_B{B}_N{N}_{'bf16' if dtype else 'f32'}", q=q, B=B, N=N, m=m, max_levels=levels,
                     min_coarse=1, dtype=dtype, act=I.RELU, head_classes=0)


def _conv(C, H, W, B, N, dtype, m=4, levels=2):
    return I.reduced(I.cfg4(1), name=f"bits_conv_c{C}_{H}x{W}_B{B}_N{N}_{'bf16' if dtype else 'f32'}", C=C, Himg=H, Wimg=W, B=B, N=N,
                     m=m, max_levels=levels, dtype=dtype, act=I.RELU)


CASES = [
    _dense(8, 3, 9, I.FP32), _dense(72, 33, 10, I.FP32), _dense(136, 130, 40, I.FP32), _dense(256, 64, 64, I.FP32),   # sweeps, lockstep
    _dense(24, 17, 9, I.BF16), _dense(200, 35, 12, I.BF16),
    _dense(128, 128, 256, I.FP32, m=2),
    _dense(264, 70, 12, I.FP32), _dense(520, 96, 16, I.BF16), _dense(512, 256, 64, I.BF16, m=2), _dense(2056, 5, 4, I.FP32, m=2),  # tiled, whole tiles, k-split
    _conv(8, 3, 5, 3, 8, I.FP32), _conv(16, 13, 11, 3, 8, I.FP32), _conv(32, 9, 7, 2, 8, I.FP32), _conv(24, 11, 3, 2, 9, I.FP32),
    _conv(48, 9, 9, 2, 6, I.FP32), _conv(16, 40, 70, 1, 4, I.FP32, m=2),                                               # lockstep; a workgroup per tap
    _conv(8, 5, 5, 2, 8, I.BF16), _conv(24, 13, 17, 5, 9, I.BF16, m=3), _conv(40, 7, 9, 3, 8, I.BF16), _conv(48, 31, 33, 1, 6, I.BF16, m=3),
    _conv(56, 9, 9, 2, 8, I.BF16), _conv(64, 16, 31, 1, 8, I.BF16), _conv(64, 23, 23, 24, 32, I.BF16, m=2, levels=3), _conv(64, 32, 32, 18, 16, I.BF16, m=2),
]


def _same(monkeypatch, run):
    monkeypatch.setenv("MGRIT_ACT_VALUES", "0")
    got = run()
    monkeypatch.setenv("MGRIT_ACT_VALUES", "1")
    ref = run()
    for a, b in zip(got, ref):
        assert np.array_equal(np.asarray(a), np.asarray(b), equal_nan=True)


@pytest.mark.parametrize("wl", CASES, ids=[w.name for w in CASES])
def test_bits_and_values_agree(wl, monkeypatch):
    print(f"\n[case] {wl.name}", flush=True)
    data = I.generate(wl)
    gp = GpuProblem(wl, data)
    rng = np.random.default_rng(5)
    U = rng.standard_normal((wl.N + 1,) + wl.state_shape).astype(np.float32)
    lam = rng.standard_normal(wl.state_shape).astype(np.float32)
    _same(monkeypatch, lambda: gp.adjoint(U, lam))


@pytest.mark.parametrize("wl", [CASES[1], CASES[12], CASES[18]], ids=lambda w: w.name)
def test_infinite_values(wl, monkeypatch):
    data = I.generate(wl)
    gp = GpuProblem(wl, data)
    U = np.random.default_rng(6).standard_normal((wl.N + 1,) + wl.state_shape).astype(np.float32)
    lam = np.ones(wl.state_shape, np.float32)
    lam.reshape(-1)[[3, -2]] = np.inf
    run = lambda: (lambda r: (r[0], r[1], r[2]))(_raw(gp, U, lam))                                  # noqa: E731
    _same(monkeypatch, run)


def _raw(gp, U, lam):
    import torch
    M = gp.M
    ws = torch.empty(M.mgrit_adjoint_workspace_bytes(gp.p), dtype=torch.uint8, device="cuda")
    Ud, l = torch.from_numpy(U).cuda(), torch.from_numpy(lam).cuda()
    Lam, dW, db = torch.zeros_like(Ud), torch.zeros(gp.W.shape, device="cuda"), torch.zeros_like(gp.b)
    M.mgrit_fas_adjoint(gp.p, gp.W, gp.b, Ud, l, Lam, dW, db, ws, check=False)
    torch.cuda.synchronize()
    return [t.cpu().numpy() for t in (Lam, dW, db)]


@pytest.mark.parametrize("dtype", [I.FP32, I.BF16], ids=["f32", "bf16"])
def test_mixed_stack(dtype, monkeypatch):
    wl = I.reduced(I.mixed(2), name="bits_mixed", B=3, C=16, Himg=6, Wimg=5, N=16, m=2, max_levels=3, fc_period=4, max_iter=2,
                   dtype=dtype, act=I.RELU)
    gp = GpuMixed(wl, I.generate(wl))
    U = np.random.default_rng(7).standard_normal((wl.N + 1,) + wl.state_shape).astype(np.float32)
    lam = np.random.default_rng(8).standard_normal(wl.state_shape).astype(np.float32)
    _same(monkeypatch, lambda: gp.adjoint(U, lam))
