"""Sweep kernels (many layer steps in one launch) at the edges of their instances, against the CPU oracle: channel counts that
fill and do not fill a block of 16, pixel counts around the multiples of 16, images that share a workgroup (the last
workgroup short), the largest image and the one past it, one coarse interval, trailing F-points, m = 2.  Every row says which
kernels its forward solve runs, S sweeps and L lockstep launches (levels with few chains of long steps), and that is checked.
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
    ("S", _conv(8, 3, 5, 3, 7, 2, 3, I.FP32)),                           # 15 pixels, half-empty channel block, m = 2, trailing
    ("S", _conv(16, 4, 4, 21, 97, 4, 2, I.FP32, act=I.RELU, it=2)),      # 16 pixels, images share workgroups, the last one short
    ("S", _conv(16, 32, 32, 1, 8, 4, 2, I.FP32)),                        # the largest image
    ("S", _conv(24, 11, 3, 2, 9, 3, 3, I.FP32, relax=I.RELAX_F)),        # 33 pixels, 24 of 32 channels
    ("S", _conv(32, 16, 32, 1, 5, 4, 2, I.FP32, act=I.RELU)),            # 512 pixels: the largest of this instance; one interval
    ("L", _conv(32, 19, 27, 1, 4, 2, 2, I.FP32)),                        # 513 pixels: lockstep launches
    ("S", _conv(16, 7, 9, 2, 4, 4, 2, I.BF16, it=2)),                    # one interval (Nc = 1)
    ("S", _conv(40, 5, 13, 2, 11, 4, 2, I.BF16)),                        # 65 pixels, 40 of 48 channels
    ("S", _conv(48, 31, 33, 1, 6, 3, 2, I.BF16, relax=I.RELAX_F)),       # 1023 pixels
    ("S", _conv(56, 8, 8, 2, 10, 2, 4, I.BF16)),                         # 56 of 64 channels
    ("S", _conv(64, 16, 32, 1, 8, 4, 2, I.BF16, act=I.RELU)),            # 512 pixels: the whole layer's weights in LDS
    ("L", _conv(64, 27, 19, 2, 18, 4, 3, I.BF16)),                       # 513 pixels, 8 chains: lockstep launches
    ("L", _conv(64, 32, 32, 1, 9, 2, 3, I.BF16, relax=I.RELAX_F, it=2)), # 1024 pixels, 4 chains: lockstep launches
    ("SL", _conv(64, 27, 19, 16, 18, 2, 2, I.BF16)),                     # 513 pixels, 144 workgroups: weights tap by tap on level 0
    # 529 pixels, 384 and 192 workgroups: weights tap by tap on levels 0 and 1, level 1 with a right-hand side of its own and
    # level 0's formed by the sweep's single steps, forward and adjoint
    ("SL", _conv(64, 23, 23, 24, 32, 2, 3, I.BF16)),
]


@pytest.mark.parametrize("kernels,wl", CONV, ids=[wl.name for _, wl in CONV])
def test_conv_sweep_instances(kernels, wl):
    print(f"\n[case] {wl.name}", flush=True)
    data = I.generate(wl)
    gp = GpuProblem(wl, data)
    gp.M.mgrit_trace_begin()
    _, U, hist, it = gp.forward()
    tr = gp.M.mgrit_trace_end()
    assert ("S" if any("sweep" in k for k in tr) else "") + ("L" if any("sweep" not in k for k in tr) else "") == kernels, tr
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
    ("S", _dense(8, 1, 7, 2, 3, I.FP32, it=2)),                          # one feature block, one row, trailing F-points
    ("S", _dense(64, 17, 12, 4, 2, I.FP32)),                             # the widest of the four-wavefront instance, 17 rows
    ("S", _dense(72, 16, 9, 3, 2, I.FP32, relax=I.RELAX_F)),             # 72 of 128 features, the last k step short
    ("S", _dense(128, 33, 5, 4, 2, I.FP32)),                             # one interval
    ("L", _dense(136, 3, 24, 2, 4, I.FP32)),                             # few chains of a wide float layer: lockstep launches
    ("SL", _dense(200, 150, 56, 4, 2, I.FP32)),                          # 140 slices of 16 rows, the last of each chain short
    ("SL", _dense(248, 400, 60, 4, 2, I.FP32, act=I.RELU)),              # 32-row slices, the last one short
    ("SL", _dense(200, 250, 32, 2, 3, I.FP32)),                          # 256 and 128 slices: level 1 too, with its right-hand side
    ("L", _dense(256, 16, 8, 4, 1, I.FP32)),                             # serial propagation of one slice: lockstep launches
    ("L", _dense(264, 5, 8, 4, 2, I.FP32)),                              # too wide: lockstep launches
    ("S", _dense(24, 40, 13, 3, 3, I.BF16)),
    ("S", _dense(104, 500, 49, 4, 2, I.BF16, it=2)),                     # 32-row slices
    ("S", _dense(256, 15, 33, 2, 3, I.BF16, relax=I.RELAX_F)),
    ("S", _dense(200, 50, 21, 5, 2, I.BF16)),
]


@pytest.mark.parametrize("kernels,wl", DENSE, ids=[wl.name for _, wl in DENSE])
def test_dense_sweep_instances(kernels, wl):
    test_conv_sweep_instances(kernels, wl)


@pytest.mark.parametrize("dtype", [I.FP32, I.BF16], ids=["fp32", "bf16"])
@pytest.mark.parametrize("q,B", [(40, 70), (40, 6130), (128, 70), (128, 6130), (168, 2040), (256, 6130)])
def test_dense_sweep_activations_elementwise(q, B, dtype, monkeypatch):
    """Four, eight and sixteen wavefronts with 16 and with 32 rows each: tanh, ReLU and the adjoint's identity (weights as
    stored and transposed), every element of two steps in sequence against float64 on the same operands."""
    gap = 0.0
    for act in (I.TANH, I.RELU):
        wl = _dense(q, B, 2, 2, 1, dtype, act=act)
        data = I.generate(wl)
        gp = GpuProblem(wl, data)
        W, b = data["W"].astype(np.float64), data["b"].astype(np.float64)
        operand = (lambda x: I.round_to_bf16(x.astype(np.float32)).astype(np.float64)) if dtype == I.BF16 else (lambda x: x.astype(np.float64))
        gp.M.mgrit_trace_begin()
        U = gp.forward()[1]
        assert any("dense_sweep" in k for k in gp.M.mgrit_trace_end())
        f = np.tanh if act == I.TANH else lambda z: np.maximum(z, 0.0)
        for n in range(2):
            ref = U[n] + wl.h * f(operand(U[n]) @ W[n].T + b[n])
            gap = max(gap, float(np.abs(U[n + 1] - ref).max()))
        lamN = np.random.default_rng(1).standard_normal(wl.state_shape).astype(np.float32)
        Uz = I.round_to_bf16(U)
        for copy in ("0", "1"):
            monkeypatch.setenv("MGRIT_ADJ_TRANSPOSED", copy)
            gp.M.mgrit_trace_begin()
            Lam = gp.adjoint(Uz, lamN, want_grad=False)[0]
            assert any("dense_sweep" in k for k in gp.M.mgrit_trace_end())
            for n in (1, 0):
                z = Uz[n].astype(np.float64) @ W[n].T + b[n]
                d = 1.0 - np.tanh(z) ** 2 if act == I.TANH else np.where(np.abs(z) < 1e-4, np.nan, (z > 0).astype(np.float64))
                if dtype == I.BF16:                                  # the cached factor and the operand are rounded
                    d = operand(d)
                x = operand((d * Lam[n + 1]).astype(np.float32)) if dtype == I.BF16 else d * Lam[n + 1]
                ref = Lam[n + 1] + wl.h * (x @ W[n])
                row = ~np.isnan(ref).any(axis=1)                     # a ReLU' decision near zero spoils its row
                assert row.mean() > 0.5
                gap = max(gap, float(np.abs(Lam[n] - ref)[row].max()))
    # float: sums of q products around 1/sqrt(q) and a state below 8, rounded to 24 bits a few times: 4e-6.  bf16: besides that
    # a rounding decided the other way, 2^-9 of one product of a weight up to 4/sqrt(q) and a value up to 4, times h
    print(f"q {q} B {B}: largest difference {gap:.2e}", flush=True)
    assert gap <= (4e-6 if dtype == I.FP32 else 0.5 / np.sqrt(q) * 4 * 4 * 2.0 ** -9 + 4e-6)


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


@pytest.mark.parametrize("relax", [I.RELAX_F, I.RELAX_FCF], ids=["F", "FCF"])
def test_a_convolution_stack_has_no_width(relax):
    """q is the width of dense stacks alone: with a value that the wide sweep takes, a convolution stack's states and history are the
    same ones."""
    wl = I.reduced(I.cfg4(2), name="conv_with_q", C=16, Himg=9, Wimg=7, B=70, N=24, m=2, max_levels=3, relax=relax)
    data, res = I.generate(wl), []
    for q in (0, 512):
        _, U, hist, _ = GpuProblem(wl, data, q=q).forward()
        res.append((U, hist))
    assert res[0][1] == res[1][1]
    assert not (res[0][0] != res[1][0]).any()
