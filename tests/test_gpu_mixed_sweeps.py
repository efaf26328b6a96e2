"""Mixed stacks whose fully connected layers open intervals: sweeps over the convolution layers between launches of the fully
connected ones.  Trailing F-points behind a fully connected layer, one interval, m = 2 (an interval of one F-point), a coarsest
level with runs of every length, both relaxations, a residual history, against the CPU oracle (relative L2 per state: float 1e-5,
bf16 operands 2e-2); infinite values against the lockstep launches."""
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
