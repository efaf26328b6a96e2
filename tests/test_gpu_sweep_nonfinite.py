"""Infinite and nearly infinite values through the sweep kernels.  They have to end as in the lockstep launches
(MGRIT_NO_SWEEP=1), which multiply float operands as they are: the same entries infinite and NaN, the rest equal to
rounding, the same status.  Serial propagation (max_levels = 1) shows every entry; a two-level solve the status."""
import numpy as np
import pytest

import mgrit_inputs as I
from tests.gpu_util import GpuProblem

pytestmark = pytest.mark.gpu

DENSE = [(24, 20, I.FP32), (24, 20, I.BF16), (72, 5, I.FP32), (128, 40, I.FP32), (136, 2048, I.FP32), (136, 20, I.BF16), (256, 33, I.BF16)]
CONV = [(16, 6, 5, 3, I.FP32), (24, 9, 7, 2, I.FP32), (40, 6, 6, 2, I.BF16)]
SHAPES = [("dense", s) for s in DENSE] + [("conv", s) for s in CONV]
IDS = [k + "_" + "x".join(str(v) for v in s[:-1]) + ("_bf16" if s[-1] else "_f32") for k, s in SHAPES]


def _workload(kind, shape, act, N, levels):
    if kind == "dense":
        q, B, dtype = shape
        return I.reduced(I.cfg5(1), name="nonfinite", q=q, B=B, N=N, m=2, max_levels=levels, min_coarse=1, dtype=dtype, act=act, head_classes=0)
    C, H, W, B, dtype = shape
    return I.reduced(I.cfg4(1), name="nonfinite", C=C, Himg=H, Wimg=W, B=B, N=N, m=2, max_levels=levels, dtype=dtype, act=act)


def _both(monkeypatch, gp, run, kernel):
    M, res = gp.M, []
    for off in (False, True):
        if off:
            monkeypatch.setenv("MGRIT_NO_SWEEP", "1")
        M.mgrit_trace_begin()
        res.append(run())
        tr = M.mgrit_trace_end()
        assert any(k.startswith(kernel) for k in tr) == (not off), tr
    monkeypatch.delenv("MGRIT_NO_SWEEP")
    return res


def _same(got, ref, tol):
    for f in (np.isnan, np.isposinf, np.isneginf):
        assert np.array_equal(f(got), f(ref)), (f.__name__, int(f(got).sum()), int(f(ref).sum()))
    ok = np.isfinite(ref)
    g, r = got[ok].astype(np.float64), ref[ok].astype(np.float64)
    assert np.linalg.norm(g - r) <= tol * np.linalg.norm(r), np.linalg.norm(g - r) / np.linalg.norm(r)


def _planted(wl, where, value):
    """One value in the last sample's state, or in the first layer's weights where the contraction index is 0."""
    data = I.generate(wl)
    if where == "state":
        data["u0"].reshape(wl.B, -1)[-1, 3] = value
        data["W"].reshape(wl.N, wl.q or wl.C, -1, wl.q or wl.C)[:, 3, :, 3] *= -np.sign(data["W"].reshape(wl.N, wl.q or wl.C, -1, wl.q or wl.C)[:, 3, :, 3])
    else:
        data["W"].reshape(wl.N, wl.q or wl.C, -1, wl.q or wl.C)[0, 5, 0, 0] = value
        data["u0"] *= np.float32(0.125)
    return data


@pytest.mark.parametrize("act", [I.RELU, I.TANH], ids=["relu", "tanh"])
@pytest.mark.parametrize("where", ["state", "weight"])
@pytest.mark.parametrize("kind,shape", SHAPES, ids=IDS)
def test_infinite_value_in_serial_propagation(kind, shape, where, act, monkeypatch):
    wl = _workload(kind, shape, act, 3, 1)
    data = _planted(wl, where, np.inf)
    gp = GpuProblem(wl, data)
    res = _both(monkeypatch, gp, lambda: gp.forward(check=False), kind + "_sweep")
    assert res[0][0] == res[1][0]
    _same(res[0][1], res[1][1], 1e-5 if wl.dtype == I.FP32 else 2e-2)


@pytest.mark.parametrize("act", [I.RELU, I.TANH], ids=["relu", "tanh"])
@pytest.mark.parametrize("where", ["state", "weight"])
@pytest.mark.parametrize("kind,shape", SHAPES, ids=IDS)
def test_infinite_value_has_the_status_of_the_lockstep_solve(kind, shape, where, act, monkeypatch):
    if kind == "dense" and shape[0] > 128 and shape[2] == I.FP32:
        pytest.skip("few chains of wide float layers run in lockstep")
    wl = _workload(kind, shape, act, 8, 2)
    data = _planted(wl, where, np.inf)
    gp = GpuProblem(wl, data)
    res = _both(monkeypatch, gp, lambda: gp.forward(check=False), kind + "_sweep")
    assert res[0][0] == res[1][0], (res[0][0], res[1][0])


@pytest.mark.parametrize("where", ["state", "weight"])
@pytest.mark.parametrize("kind,shape", SHAPES, ids=IDS)
def test_infinite_value_in_the_serial_adjoint(kind, shape, where, monkeypatch):
    """Weights as stored (contraction over their slow index) in the dense kernels."""
    wl = _workload(kind, shape, I.RELU, 3, 1)
    data = _planted(wl, "state", 0.5)
    U = np.stack([data["u0"]] * (wl.N + 1))
    lamN = np.random.default_rng(2).standard_normal(wl.state_shape).astype(np.float32)
    if where == "state":
        lamN.reshape(wl.B, -1)[-1, 3] = np.inf
    else:
        data["W"].reshape(wl.N, wl.q or wl.C, -1, wl.q or wl.C)[1, 0, 0, 5] = np.inf
    gp = GpuProblem(wl, data)
    res = _both(monkeypatch, gp, lambda: gp.adjoint(U, lamN, want_grad=False)[0], kind + "_sweep")
    _same(res[0], res[1], 1e-5 if wl.dtype == I.FP32 else 2e-2)


@pytest.mark.parametrize("act", [I.RELU, I.TANH], ids=["relu", "tanh"])
@pytest.mark.parametrize("where", ["state", "weight"])
@pytest.mark.parametrize("kind,shape", [(k, s) for k, s in SHAPES if s[-1] == I.FP32], ids=[i for i, (k, s) in zip(IDS, SHAPES) if s[-1] == I.FP32])
def test_largest_floats_stay_finite(kind, shape, where, act, monkeypatch):
    """Finite values above the largest bf16 number, 3.39e38, in one layer step."""
    wl = _workload(kind, shape, act, 1, 1)
    data = _planted(wl, where, np.float32(3.4e38))
    data["u0"] = np.where(data["u0"] > 1e38, data["u0"], np.clip(data["u0"], -0.9, 0.9)).astype(np.float32)
    gp = GpuProblem(wl, data)
    res = _both(monkeypatch, gp, lambda: gp.forward(check=False), kind + "_sweep")
    assert np.isfinite(res[1][1]).all()
    _same(res[0][1], res[1][1], 1e-5)


@pytest.mark.parametrize("relax", [I.RELAX_F, I.RELAX_FCF], ids=["F", "FCF"])
@pytest.mark.parametrize("kind,shape", [("dense", (24, 20, I.FP32)), ("dense", (128, 40, I.FP32)), ("dense", (136, 600, I.FP32)),
                                        ("conv", (16, 6, 5, 3, I.FP32)), ("conv", (24, 9, 7, 2, I.FP32))])
def test_whole_solves_with_a_weight_that_does_not_split(kind, shape, relax, monkeypatch):
    """Through tanh a weight of 3.4e38 leaves finite states, so every array of a solve that repeated chains write can be
    compared: relaxation, coarse right-hand side and its norm, coarse solve, closing sweep with trailing F-points."""
    wl = I.reduced(_workload(kind, shape, I.TANH, 19, 3), relax=relax, max_iter=2)
    data = _planted(wl, "weight", np.float32(3.4e38))
    gp = GpuProblem(wl, data)
    fwd = _both(monkeypatch, gp, lambda: gp.forward(), kind + "_sweep")
    _same(fwd[0][1], fwd[1][1], 1e-5)
    for a, b in zip(fwd[0][2], fwd[1][2]):
        assert abs(a - b) <= 1e-4 * b, (fwd[0][2], fwd[1][2])
    lamN = np.random.default_rng(6).standard_normal(wl.state_shape).astype(np.float32)
    adj = _both(monkeypatch, gp, lambda: gp.adjoint(fwd[1][1], lamN), kind + "_sweep")
    for x, y in zip(adj[0][:3], adj[1][:3]):
        assert np.isfinite(y).all()
        _same(x, y, 1e-5)
