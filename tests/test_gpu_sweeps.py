"""Sweep kernels (many layer steps in one launch) at the edges of their instances, against the CPU oracle: channel counts that
fill and do not fill a block of 16, pixel counts around the multiples of 16, images that share a workgroup (the last
workgroup short), the largest image and the one past it, one coarse interval, trailing F-points, m = 2.
Tolerances (relative L2 per state / per layer gradient): float 1e-5, bf16 operands 2e-2, as in the other parity tests."""
import numpy as np
import pytest

import mgrit_inputs as I
from tests.gpu_util import GpuProblem, oracle_forward, oracle_adjoint, rel_l2_per_state

pytestmark = pytest.mark.gpu
TOL = {I.FP32: 1e-5, I.BF16: 2e-2}


def _conv(C, H, W, B, N, m, levels, dtype, relax=I.RELAX_FCF, act=I.TANH, it=1):
    name = f"sweep_conv_c{C}_{H}x{W}_B{B}_N{N}_m{m}_L{levels}_{'bf16' if dtype else 'fp32'}_{'FCF' if relax else 'F'}_{'relu' if act else 'tanh'}"
    return I.reduced(I.cfg4(it), name=name, C=C, Himg=H, Wimg=W, B=B, N=N, m=m, max_levels=levels, dtype=dtype, relax=relax, act=act)


CONV = [
    _conv(8, 3, 5, 3, 7, 2, 3, I.FP32),                            # 15 pixels, half-empty channel block, m = 2, trailing
    _conv(16, 4, 4, 21, 97, 4, 2, I.FP32, act=I.RELU, it=2),       # 16 pixels, images share workgroups, the last one short
    _conv(16, 32, 32, 1, 8, 4, 2, I.FP32),                         # the largest image
    _conv(24, 11, 3, 2, 9, 3, 3, I.FP32, relax=I.RELAX_F),         # 33 pixels, 24 of 32 channels
    _conv(32, 16, 32, 1, 5, 4, 2, I.FP32, act=I.RELU),             # 512 pixels: the largest of this instance; one interval
    _conv(32, 19, 27, 1, 4, 2, 2, I.FP32),                         # 513 pixels: lockstep launches
    _conv(16, 7, 9, 2, 4, 4, 2, I.BF16, it=2),                     # one interval (Nc = 1)
    _conv(40, 5, 13, 2, 11, 4, 2, I.BF16),                         # 65 pixels, 40 of 48 channels
    _conv(48, 31, 33, 1, 6, 3, 2, I.BF16, relax=I.RELAX_F),        # 1023 pixels
    _conv(56, 8, 8, 2, 10, 2, 4, I.BF16),                          # 56 of 64 channels
    _conv(64, 16, 32, 1, 8, 4, 2, I.BF16, act=I.RELU),             # 512 pixels: the whole layer's weights in LDS
    _conv(64, 27, 19, 2, 18, 4, 3, I.BF16),                        # 513 pixels: weights tap by tap
    _conv(64, 32, 32, 1, 9, 2, 3, I.BF16, relax=I.RELAX_F, it=2),  # 1024 pixels
    _conv(64, 27, 19, 16, 18, 2, 2, I.BF16),                       # 513 pixels, 144 workgroups: weights tap by tap
]


@pytest.mark.parametrize("wl", CONV, ids=lambda w: w.name)
def test_conv_sweep_instances(wl):
    print(f"\n[case] {wl.name}", flush=True)
    data = I.generate(wl)
    gp = GpuProblem(wl, data)
    _, U, hist, it = gp.forward()
    Uo, hist_o, it_o = oracle_forward(wl, data)
    tol = TOL[wl.dtype]
    assert it == it_o and rel_l2_per_state(U, Uo) <= tol
    # a residual that has converged stops at the float32 rounding floor: one ulp of the largest state value per entry
    sizes, _ = gp.M.mgrit_level_map(gp.p)
    floor = 2.0 ** -23 * float(np.abs(Uo).max()) * np.sqrt((sizes[min(1, len(sizes) - 1)] + 1) * wl.E)
    for a, b in zip(hist, hist_o):
        assert abs(a - b) <= (1e-3 if wl.dtype == I.FP32 else 0.2) * b + floor, (hist, hist_o)
    if wl.dtype == I.FP32 and wl.act == I.RELU:
        return                                   # ReLU' is a 0/1 decision that summation order can turn
    Ul = Uo.astype(np.float32) if wl.dtype == I.FP32 else I.round_to_bf16(Uo.astype(np.float32))
    lamN = np.random.default_rng(3).standard_normal(wl.state_shape).astype(np.float32)
    Lam, dW, db, _, _ = gp.adjoint(Ul, lamN)
    Lo, dWo, dbo, _, _ = oracle_adjoint(wl, data, Ul, lamN)
    eL, eW, eb = rel_l2_per_state(Lam, Lo), rel_l2_per_state(dW, dWo), rel_l2_per_state(db, dbo)
    print(f"{wl.name}: Lam {eL:.2e} dW {eW:.2e} db {eb:.2e}", flush=True)
    assert eL <= tol and eW <= tol and eb <= tol, (eL, eW, eb)


def _dense(q, B, N, m, levels, dtype, relax=I.RELAX_FCF, act=I.TANH, it=1):
    name = f"sweep_dense_q{q}_B{B}_N{N}_m{m}_L{levels}_{'bf16' if dtype else 'fp32'}_{'FCF' if relax else 'F'}_{'relu' if act else 'tanh'}"
    return I.reduced(I.cfg5(it), name=name, q=q, B=B, N=N, m=m, max_levels=levels, min_coarse=1, dtype=dtype, relax=relax, act=act,
                     head_classes=0)


DENSE = [
    _dense(8, 1, 7, 2, 3, I.FP32, it=2),                           # one feature block, one row, trailing F-points
    _dense(64, 17, 12, 4, 2, I.FP32),                              # the widest of the four-wavefront instance, 17 rows
    _dense(72, 16, 9, 3, 2, I.FP32, relax=I.RELAX_F),              # 72 of 128 features, the last k step short
    _dense(128, 33, 5, 4, 2, I.FP32),                              # one interval
    _dense(136, 3, 24, 2, 4, I.FP32),                              # 136 of 256
    _dense(200, 150, 56, 4, 2, I.FP32),                            # 140 slices of 16 rows, the last of each chain short
    _dense(248, 400, 60, 4, 2, I.FP32, act=I.RELU),                # 32-row slices, the last one short
    _dense(256, 16, 8, 4, 1, I.FP32),                              # serial propagation
    _dense(264, 5, 8, 4, 2, I.FP32),                               # too wide: lockstep launches
    _dense(24, 40, 13, 3, 3, I.BF16),
    _dense(104, 500, 49, 4, 2, I.BF16, it=2),                      # 32-row slices
    _dense(256, 15, 33, 2, 3, I.BF16, relax=I.RELAX_F),
    _dense(200, 50, 21, 5, 2, I.BF16),
]


@pytest.mark.parametrize("wl", DENSE, ids=lambda w: w.name)
def test_dense_sweep_instances(wl):
    test_conv_sweep_instances(wl)


@pytest.mark.parametrize("C,H,W", [(16, 8, 8), (64, 8, 8)])
def test_bf16_convolution_residual_reaches_rounding(C, H, W):
    """After as many cycles as there are intervals FAS is exact, and the C-points' residual is what the two roundings of
    (P - Phi) + Phi leave: 2^-22 of the largest value per entry.  It needs both coarse steps to round alike."""
    wl = _conv(C, H, W, 4, 32, 4, 2, I.BF16, it=9)
    gp = GpuProblem(wl, I.generate(wl))
    _, U, hist, _ = gp.forward()
    sizes, _ = gp.M.mgrit_level_map(gp.p)
    bound = 2.0 ** -22 * float(np.abs(U).max()) * np.sqrt((sizes[1] + 1) * wl.E)
    print(hist, bound, flush=True)
    assert hist[-1] <= bound


# the smallest number of chains that a long step is worth a sweep for, and one less: serial propagation (max_levels = 1), where
# an image or 16 rows are a chain's workgroup; one instance of every other kind with a single chain
EDGES = [(_conv(64, 28, 28, 127, 2, 2, 1, I.BF16), "forward", False), (_conv(64, 28, 28, 128, 2, 2, 1, I.BF16), "forward", True),
         (_conv(64, 28, 28, 143, 2, 2, 1, I.BF16), "adjoint", False), (_conv(64, 28, 28, 144, 2, 2, 1, I.BF16), "adjoint", True),
         (_conv(64, 23, 23, 191, 2, 2, 1, I.BF16), "adjoint", False), (_conv(64, 23, 23, 192, 2, 2, 1, I.BF16), "adjoint", True),
         (_conv(48, 31, 31, 31, 3, 2, 1, I.BF16), "adjoint", False), (_conv(48, 31, 31, 32, 3, 2, 1, I.BF16), "adjoint", True),
         (_conv(48, 30, 30, 1, 3, 2, 1, I.BF16), "adjoint", True), (_conv(48, 32, 32, 1, 3, 2, 1, I.BF16), "forward", True),
         (_conv(32, 20, 30, 1, 3, 2, 1, I.BF16), "adjoint", True), (_conv(24, 32, 32, 2, 3, 2, 1, I.BF16), "adjoint", True),
         (_conv(56, 16, 32, 1, 3, 2, 1, I.BF16), "adjoint", True), (_conv(56, 19, 27, 1, 3, 2, 1, I.BF16), "forward", False),
         (_conv(32, 16, 32, 1, 3, 2, 1, I.FP32), "adjoint", True)]


@pytest.mark.parametrize("wl,direction,sweep", EDGES, ids=lambda v: v if isinstance(v, str) else getattr(v, "name", None))
def test_kernel_choice_at_the_edges_of_its_rule(wl, direction, sweep, monkeypatch):
    """Which kernel runs, and that both kernels give the same result there."""
    print(f"\n[case] {wl.name} {direction}", flush=True)
    data = I.generate(wl)
    gp = GpuProblem(wl, data)
    rng = np.random.default_rng(4)
    U = rng.standard_normal((wl.N + 1,) + wl.state_shape).astype(np.float32)
    lamN = rng.standard_normal(wl.state_shape).astype(np.float32)
    run = (lambda: gp.forward()[1]) if direction == "forward" else (lambda: gp.adjoint(U, lamN, want_grad=False)[0])
    gp.M.mgrit_trace_begin()
    got = run()
    tr = gp.M.mgrit_trace_end()
    kernel = "conv_sweep_kernel" if wl.layer == I.CONV else "dense_sweep_kernel"
    assert any(k.startswith(kernel) for k in tr) == sweep, tr
    monkeypatch.setenv("MGRIT_NO_SWEEP", "1")
    assert rel_l2_per_state(got, run()) <= (1e-6 if wl.dtype == I.FP32 else 1e-3)      # the same operands, sums in another order
