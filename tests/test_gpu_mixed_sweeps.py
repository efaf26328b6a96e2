"""Mixed stacks whose fully connected layers open intervals: sweeps over the convolution layers between launches of the fully
connected ones.  Trailing F-points behind a fully connected layer, one interval, m = 2 (an interval of one F-point), a coarsest
level with runs of every length, both relaxations, a residual history, against the CPU oracle (relative L2 per state: float 1e-5,
bf16 operands 2e-2); infinite values, weights that have no bf16 parts and samples that share a workgroup with infinite ones against
the lockstep launches, entry by entry where differences of infinite values take no part."""
import numpy as np
import pytest

import mgrit_inputs as I
from tests.gpu_util import rel_l2_per_state
from tests.test_gpu_mixed import GpuMixed, _mx, _oracle_forward

pytestmark = pytest.mark.gpu

CASES = [
    _mx("msweep_c16_P8_N23_m2_L3", N=23, fc_period=8),
    _mx("msweep_c8_P16_N69_m4_L2_F", C=8, Himg=5, Wimg=4, N=69, m=4, max_levels=2, fc_period=16, relax=I.RELAX_F),
    _mx("msweep_c16_P6_N8_m3_L2_one_interval", Himg=4, Wimg=4, N=5, m=3, max_levels=2, fc_period=6),
    _mx("msweep_c16_P4_N64_m4_L3_every_interval", Himg=4, Wimg=4, B=5, N=64, m=4, fc_period=4),
    _mx("msweep_c24_bf16_P12_N50_m3_L3", dtype=I.BF16, C=24, Himg=6, Wimg=6, N=50, m=3, fc_period=12, act=I.TANH),
    _mx("msweep_c16_P5_N13_serial", Himg=4, Wimg=4, N=13, max_levels=1, fc_period=5, max_iter=1),
]


@pytest.mark.parametrize("wl", CASES, ids=[w.name for w in CASES])
def test_against_the_oracle(wl):
    print(f"\n[case] {wl.name}", flush=True)
    data = I.generate(wl)
    gm = GpuMixed(wl, data)
    gm.M.mgrit_trace_begin()
    U, hist, it = gm.forward()
    tr = gm.M.mgrit_trace_end()
    assert "conv_sweep_kernel" in tr, tr
    Uo, hist_o, it_o = _oracle_forward(wl, data)
    assert it == it_o and rel_l2_per_state(U, Uo) <= (1e-5 if wl.dtype == I.FP32 else 2e-2)
    floor = 2.0 ** -23 * float(np.abs(Uo).max()) * np.sqrt((wl.N // wl.m + 1) * wl.E)
    assert all(abs(a - b) <= (1e-3 if wl.dtype == I.FP32 else 0.2) * b + floor for a, b in zip(hist, hist_o)), (hist, hist_o)


@pytest.mark.parametrize("wl", [CASES[0], CASES[5]], ids=["levels", "serial"])
def test_infinite_values_as_in_lockstep_launches(wl, monkeypatch):
    """Every entry of a serial propagation; of a multilevel solve, where differences of infinite values take part, the status."""
    import torch
    data = I.generate(wl)
    data["u0"].reshape(wl.B, -1)[-1, 3] = np.inf
    gm, res, status = GpuMixed(wl, data), [], []
    for off in (False, True):
        if off:
            monkeypatch.setenv("MGRIT_NO_SWEEP", "1")
        status.append(gm.M.mgrit_fas_forward_mixed(gm.p, gm.fc, gm.W, gm.b, gm.u0, gm.U, gm.ws, check=False)[0])
        torch.cuda.synchronize()
        res.append(gm.U.cpu().numpy())
    assert status[0] == status[1]
    if wl.max_levels == 1:
        for f in (np.isnan, np.isposinf, np.isneginf):
            assert np.array_equal(f(res[0]), f(res[1])), f.__name__


def _sweeps_and_lockstep(gm, monkeypatch):
    """States and history of the solve with sweeps, then of the one without."""
    import torch
    res = []
    for off in (False, True):
        if off:
            monkeypatch.setenv("MGRIT_NO_SWEEP", "1")
        gm.U.fill_(float("nan"))
        gm.M.mgrit_trace_begin()
        _, hist, _ = gm.M.mgrit_fas_forward_mixed(gm.p, gm.fc, gm.W, gm.b, gm.u0, gm.U, gm.ws, check=False)
        torch.cuda.synchronize()
        assert ("conv_sweep_kernel" in gm.M.mgrit_trace_end()) == (not off)
        res.append((gm.U.cpu().numpy(), hist))
    return res


@pytest.mark.parametrize("relax", [I.RELAX_F, I.RELAX_FCF], ids=["F", "FCF"])
@pytest.mark.parametrize("m,P,N,layer", [(2, 8, 43, 1), (2, 8, 43, 9), (2, 8, 43, 2), (2, 8, 43, 10), (4, 16, 69, 3), (4, 16, 69, 34), (3, 9, 40, 20)])
def test_whole_solves_with_a_weight_that_does_not_split(m, P, N, layer, relax, monkeypatch):
    """As in plain stacks: through tanh a weight of 3.4e38 leaves finite states, and every array that repeated chains write can be
    compared.  The layer is in an interval that a fully connected one opens, the first or a later one, of level 0 or also of level 1."""
    wl = _mx("msweep_split", Himg=4, Wimg=4, N=N, m=m, fc_period=P, relax=relax, act=I.TANH)
    data = I.generate(wl)
    data["W"].reshape(N, wl.C, -1, wl.C)[layer, 5, 0, 0] = np.float32(3.4e38)
    data["u0"] *= np.float32(0.125)
    (U, hist), (Ur, hist_r) = _sweeps_and_lockstep(GpuMixed(wl, data), monkeypatch)
    assert np.isfinite(Ur).all() and rel_l2_per_state(U, Ur) <= 1e-5
    for a, b in zip(hist, hist_r):
        assert abs(a - b) <= 1e-4 * b, (hist, hist_r)


@pytest.mark.parametrize("relax", [I.RELAX_F, I.RELAX_FCF], ids=["F", "FCF"])
def test_samples_beside_an_infinite_one(relax, monkeypatch):
    """Four images of 4 x 4 pixels share a workgroup; one of them starts with an infinite value."""
    wl = _mx("msweep_shared", Himg=4, Wimg=4, B=16, N=128, m=2, fc_period=8, relax=relax, act=I.TANH)
    data = I.generate(wl)
    data["u0"].reshape(wl.B, -1)[5, 3] = np.inf
    (U, _), (Ur, _) = _sweeps_and_lockstep(GpuMixed(wl, data), monkeypatch)
    others = [i for i in range(wl.B) if i != 5]
    assert np.isfinite(Ur[:, others]).all() and rel_l2_per_state(U[:, others], Ur[:, others]) <= 1e-5
