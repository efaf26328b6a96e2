"""Dense layers of width 8 and 16: one wavefront per slice of 16 rows and chain, sweeps that follow one another in one launch.
Against the CPU oracle: slices that are not full, more chains than a workgroup has wavefronts (some sweeps then have a launch of
their own), more sweeps than a launch holds, trailing F-points, every start, a run to a tolerance; and against the lockstep
launches (MGRIT_NO_SWEEP=1) where values are infinite.  Tolerances (relative L2 per state / layer gradient): float 1e-5, bf16
operands 2e-2, as in the other parity tests."""
import numpy as np
import pytest

import mgrit_inputs as I
from tests.gpu_util import GpuProblem, oracle_forward, oracle_adjoint, rel_l2_per_state

pytestmark = pytest.mark.gpu
TOL = {I.FP32: 1e-5, I.BF16: 2e-2}


def _dense(q, B, N, m, levels, dtype, relax=I.RELAX_FCF, it=2, act=I.TANH):
    name = f"narrow_q{q}_B{B}_N{N}_m{m}_L{levels}_{'bf16' if dtype else 'f32'}_{'FCF' if relax else 'F'}_it{it}"
    return I.reduced(I.cfg5(it), name=name, q=q, B=B, N=N, m=m, max_levels=levels, min_coarse=1, dtype=dtype, relax=relax, act=act, head_classes=0)


CASES = [
    _dense(8, 1, 16, 4, 2, I.FP32), _dense(16, 16, 17, 2, 3, I.FP32, relax=I.RELAX_F), _dense(16, 17, 79, 4, 3, I.FP32),
    _dense(8, 33, 203, 3, 4, I.FP32, it=3), _dense(16, 40, 64, 2, 6, I.FP32, it=4), _dense(8, 5, 7, 2, 1, I.FP32, it=1),
    _dense(16, 300, 260, 2, 2, I.FP32, it=1), _dense(8, 20, 31, 3, 3, I.BF16), _dense(16, 50, 130, 4, 3, I.BF16, relax=I.RELAX_F, act=I.RELU),
    _dense(16, 3, 12, 4, 2, I.BF16),
]


@pytest.mark.parametrize("wl", CASES, ids=[w.name for w in CASES])
def test_against_the_oracle(wl):
    print(f"\n[case] {wl.name}", flush=True)
    data = I.generate(wl)
    gp = GpuProblem(wl, data)
    gp.M.mgrit_trace_begin()
    _, U, hist, it = gp.forward()
    tr = gp.M.mgrit_trace_end()
    assert tr and all("sweep" in k for k in tr), tr
    Uo, hist_o, it_o = oracle_forward(wl, data)
    tol = TOL[wl.dtype]
    assert it == it_o and rel_l2_per_state(U, Uo) <= tol
    sizes, _ = gp.M.mgrit_level_map(gp.p)
    floor = 2.0 ** -23 * float(np.abs(Uo).max()) * np.sqrt((sizes[min(1, len(sizes) - 1)] + 1) * wl.E)
    for a, b in zip(hist, hist_o):
        assert abs(a - b) <= (1e-3 if wl.dtype == I.FP32 else 0.2) * b + floor, (hist, hist_o)
    if wl.act == I.RELU:
        return                                   # ReLU' is a 0/1 decision that summation order can turn
    lamN = np.random.default_rng(1).standard_normal(wl.state_shape).astype(np.float32)
    Lam, dW, db, _, _ = gp.adjoint(U, lamN)
    Lo, dWo, dbo, _, _ = oracle_adjoint(wl, data, U.astype(np.float64), lamN)
    assert rel_l2_per_state(Lam, Lo) <= tol
    assert np.linalg.norm(dW - dWo) <= tol * np.linalg.norm(dWo) and np.linalg.norm(db - dbo) <= tol * np.linalg.norm(dbo)


@pytest.mark.parametrize("init", [0, 1, 2, 3], ids=["zero", "copy", "user", "nested"])
@pytest.mark.parametrize("tol", [0.0, 1e-5])
def test_starts_and_tolerance(init, tol):
    """Collected sweeps around the launches that are not sweeps (clearing, a norm read on the host): both relaxations, three levels."""
    for relax in (I.RELAX_F, I.RELAX_FCF):
        wl = _dense(16, 21, 50, 3, 3, I.FP32, relax=relax, it=6 if tol else 2)
        data = I.generate(wl)
        gp = GpuProblem(wl, data, init=init, tol=tol, norm_kind=1)
        U0 = np.random.default_rng(2).standard_normal((wl.N + 1,) + wl.state_shape).astype(np.float32) if init == 2 else None
        _, U, hist, it = gp.forward(U_init=U0)
        Uo, hist_o, it_o = oracle_forward(wl, data, init=init, U_init=U0, tol=tol, norm_kind=1)
        assert it == it_o and rel_l2_per_state(U, Uo) <= 1e-5
        assert all(abs(a - b) <= 1e-3 * b + 2e-7 for a, b in zip(hist, hist_o)), (hist, hist_o)


@pytest.mark.parametrize("dtype", [I.FP32, I.BF16], ids=["f32", "bf16"])
@pytest.mark.parametrize("q", [8, 16])
def test_infinite_values_as_in_lockstep_launches(q, dtype, monkeypatch):
    import torch
    wl = _dense(q, 19, 6, 2, 1, dtype, it=1, act=I.RELU)
    data = I.generate(wl)
    data["u0"].reshape(wl.B, -1)[-1, 3] = np.inf
    data["W"][2, 5, 0] = np.inf if dtype == I.FP32 else data["W"][2, 5, 0]
    gp, res = GpuProblem(wl, data), []
    for off in (False, True):
        if off:
            monkeypatch.setenv("MGRIT_NO_SWEEP", "1")
        gp.M.mgrit_fas_forward(gp.p, gp.W, gp.b, gp.u0, gp.U, gp.ws, check=False)
        torch.cuda.synchronize()
        res.append(gp.U.cpu().numpy())
    got, ref = res
    for f in (np.isnan, np.isposinf, np.isneginf):
        assert np.array_equal(f(got), f(ref)), f.__name__
    ok = np.isfinite(ref)
    assert np.abs(got[ok] - ref[ok]).max() <= (1e-5 if dtype == I.FP32 else 2e-2) * np.abs(ref[ok]).max()
