"""The parameter gradient of float convolution layers of at most 32 channels, whose operands are three bf16 parts: against 64 bits
about the multipliers that the same call returned, at slabs of one row and of whole images, widths around multiples of eight, fewer
slabs than chunks and more, channel counts that fill a block of 16, half of it and one and a half; and with values that have no
such parts (infinite ones, finite ones above 3.396e38), where the sums are formed again from the floats."""
import numpy as np
import pytest

import mgrit_inputs as I
from tests.gpu_util import GpuProblem
from tests.test_gpu_relu_factors import _raw

pytestmark = pytest.mark.gpu


def _wl(C, H, W, B, N, act=I.RELU):
    return I.reduced(I.cfg4(1), name=f"cgrad_c{C}_{H}x{W}_B{B}_N{N}_{'relu' if act == I.RELU else 'tanh'}", C=C, Himg=H, Wimg=W, B=B, N=N,
                     m=2, max_levels=2, dtype=I.FP32, act=act)


CASES = [_wl(*c) for c in ((8, 1, 1, 1, 4), (8, 5, 3, 2, 4), (8, 28, 28, 3, 4), (16, 7, 8, 3, 4), (16, 13, 9, 2, 5, I.TANH), (16, 28, 28, 2, 3),
                           (16, 4, 64, 2, 2), (16, 9, 33, 3, 300), (16, 32, 32, 1, 2, I.TANH), (24, 13, 17, 2, 4), (32, 16, 16, 2, 3),
                           (32, 3, 64, 1, 2), (32, 31, 25, 2, 2, I.TANH))]


def _shifted(u):
    """u [B, H, W, C] -> the nine shifted copies [3, 3, B, H, W, C], zeros around the images."""
    p = np.pad(u, ((0, 0), (1, 1), (1, 1), (0, 0)))
    H, W = u.shape[1:3]
    return np.stack([np.stack([p[:, y:y + H, x:x + W] for x in range(3)]) for y in range(3)])


def _exact(wl, data, U, Lam):
    """dW, db and the sums of the absolute products behind them, in 64 bits; G's error where act' is rounded."""
    out = [np.zeros((wl.N, wl.C, 3, 3, wl.C)), np.zeros((wl.N, wl.C))]
    mag = [np.zeros_like(o) for o in out]
    with np.errstate(invalid="ignore", over="ignore"):
        for n in range(wl.N):
            S = _shifted(U[n].astype(np.float64))
            K = data["W"][n].astype(np.float64)
            z = sum((S[y, x].reshape(-1, wl.C) @ K[:, y, x].T for y in range(3) for x in range(3))) + data["b"][n]
            D = (z > 0).astype(np.float64) if wl.act == I.RELU else 1.0 - np.tanh(z) ** 2
            G = wl.h * D * Lam[n + 1].astype(np.float64).reshape(-1, wl.C)
            A = np.abs(wl.h * Lam[n + 1].astype(np.float64).reshape(-1, wl.C)) if wl.act != I.RELU else np.abs(G)
            for y in range(3):
                for x in range(3):
                    s = S[y, x].reshape(-1, wl.C)
                    if np.isfinite(s).all():
                        out[0][n, :, y, x], mag[0][n, :, y, x] = G.T @ s, A.T @ np.abs(s)
                    else:                                       # (product by product: a library's sums may skip or reorder)
                        out[0][n, :, y, x] = (G[:, :, None] * s[:, None, :]).sum(0)
            out[1][n], mag[1][n] = G.sum(0), A.sum(0)
    return out, mag


def _inputs(wl, seed):
    rng = np.random.default_rng(seed)
    U = rng.standard_normal((wl.N + 1,) + wl.state_shape).astype(np.float32)
    return U, rng.standard_normal(wl.state_shape).astype(np.float32)


@pytest.mark.parametrize("wl", CASES, ids=[w.name for w in CASES])
def test_against_64_bits(wl):
    print(f"\n[case] {wl.name}", flush=True)
    data = I.generate(wl)
    U, lam = _inputs(wl, 3)
    Lam, dW, db = _raw(GpuProblem(wl, data), U, lam)
    ref, mag = _exact(wl, data, U, Lam)
    # of the sum of absolute products: 2^-24 each for the product G is, the factor h and the parts left out, twice one for the last
    # additions of partial sums, and one for every addition of 32 products to a sum; act' of tanh is good to 1e-6
    steps = -(-wl.B * wl.Himg * ((wl.Wimg + 7) & ~7) // 32) + 2 * wl.B * wl.Himg
    tol = 2.0 ** -24 * (8 + steps) + (1e-6 if wl.act == I.TANH else 0.0)
    for got, r, m in zip((dW, db), ref, mag):
        assert (np.abs(got.reshape(r.shape) - r) <= tol * m + 1e-30).all()


@pytest.mark.parametrize("su,sl", [(1.0, 1e-34), (1.0, 1e-36), (1.0, 1e-37), (1e-37, 1.0), (1e-18, 1e-18), (0.0, 1.0)])
@pytest.mark.parametrize("wl", [CASES[1], CASES[3], CASES[9], CASES[12]], ids=lambda w: w.name)
def test_values_whose_lower_parts_are_too_small(wl, su, sl):
    """States or multipliers so small that bf16 has no numbers for their lower parts: the same accuracy, but for sums that are
    themselves rounded to multiples of 2^-149."""
    data = I.generate(wl)
    U, lam = _inputs(wl, 5)
    Lam, dW, db = _raw(GpuProblem(wl, data), U * np.float32(su), lam * np.float32(sl))
    ref, mag = _exact(wl, data, U * np.float32(su), Lam)
    n = wl.B * wl.Himg * wl.Wimg
    steps = -(-wl.B * wl.Himg * ((wl.Wimg + 7) & ~7) // 32) + 2 * wl.B * wl.Himg
    tol = 2.0 ** -24 * (8 + steps) + (1e-6 if wl.act == I.TANH else 0.0)
    for got, r, m in zip((dW, db), ref, mag):
        assert (np.abs(got.reshape(r.shape) - r) <= tol * m + 4 * n * 2.0 ** -149).all()


@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan, 3.4e38], ids=["inf", "-inf", "nan", "3.4e38"])
@pytest.mark.parametrize("wl", [CASES[2], CASES[3], CASES[5], CASES[7], CASES[9], CASES[10], CASES[12]], ids=lambda w: w.name)
def test_values_without_parts(wl, value, monkeypatch):
    data = I.generate(wl)
    U, lam = _inputs(wl, 4)
    U[1, 0, 2, 3, 5] = value
    U[0, -1, wl.Himg - 1, wl.Wimg - 1, 0] = value
    gp = GpuProblem(wl, data)
    Lam, dW, db = _raw(gp, U, lam * np.float32(1e-3))
    (rW, rb), _ = _exact(wl, data, U, Lam)
    for got, r in ((dW, rW), (db, rb)):
        got = got.reshape(r.shape)
        assert np.array_equal(np.isnan(got), np.isnan(r)) and np.array_equal(np.isinf(got), np.isinf(r))
        assert np.array_equal(np.sign(got[np.isinf(r)]), np.sign(r[np.isinf(r)]))
        ok = np.isfinite(r)
        assert np.linalg.norm((got[ok] / 1e30) - (r[ok] / 1e30)) <= 1e-5 * np.linalg.norm(r[ok] / 1e30)


@pytest.mark.parametrize("C,H,W,B", [(8, 28, 28, 16), (16, 28, 28, 16), (32, 30, 32, 8)])
def test_values_without_parts_do_not_stall_the_gradient(C, H, W, B):
    """A NaN in every layer's states: the sums formed again take a few times as long, not a hundred.  (Measured 4 to 7 times; with
    a thread per output that walks the pixels in global memory 45 to 180.)"""
    import torch
    import paper_2007_07336_amd as M
    N = 32
    p = M.make_problem(N=N, h=1.0 / N, m=4, max_levels=2, min_coarse=1, relax=0, max_iter=1, layer=1, act=1, dtype=0, B=B, C=C, Himg=H, Wimg=W)
    g = torch.Generator(device="cuda").manual_seed(C)
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda")                                     # noqa: E731
    Wt, b, U, lam = rnd(N, C, 3, 3, C), rnd(N, C), rnd(N + 1, B, H, W, C), rnd(B, H, W, C)
    Lam, dW, db = torch.empty_like(U), torch.empty_like(Wt), torch.empty_like(b)
    ws = torch.empty(M.mgrit_adjoint_workspace_bytes(p), dtype=torch.uint8, device="cuda")

    def gradient_us():
        """of the shortest of five solves, less those without a gradient"""
        times = []
        for w, d in ((dW, db), (None, None)):
            one = []
            for _ in range(6):
                t0, t1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
                t0.record()
                M.mgrit_fas_adjoint(p, Wt, b, U, lam, Lam, w, d, ws, want_hist=False, check=False)
                t1.record()
                torch.cuda.synchronize()
                one.append(1e3 * t0.elapsed_time(t1))
            times.append(min(one[1:]))
        return times[0] - times[1]
    finite = gradient_us()
    U[:, 0, 0, 0, 0] = float("nan")
    bad = gradient_us()
    print(f"\nC{C}: {finite:.0f} us, {bad:.0f} with a NaN", flush=True)
    assert bool(torch.isnan(dW).any()) and bad <= 20 * max(finite, 20.0)
