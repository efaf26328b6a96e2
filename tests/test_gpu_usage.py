"""GPU tests of the path used the way the paper uses it (Sec. IV-A, IV-C): early-stopped forward and
adjoint solves drive a gradient-descent loop.  The head (softmax cross-entropy on u^N) and the parameter
update are plain torch on the device; every layer step, adjoint step and parameter gradient runs in the
library.  Synthetic inputs and labels."""
import numpy as np
import pytest

import mgrit_inputs as I
from oracle import mgrit_oracle as O
from tests.gpu_util import GpuProblem, rel_l2_per_state

pytestmark = pytest.mark.gpu


def _say(msg):
    print(f"\n[case] {msg}", flush=True)


def test_solve_on_a_side_stream_matches_default_stream():
    """All work goes to the stream handed over: a solve on a non-default stream, overlapped with unrelated work
    on the default stream, gives bitwise the same result as on the default stream."""
    import torch
    import paper_2007_07336_amd as M
    wl = I.reduced(I.cfg2(2), name="dense_fp32_side_stream", q=72, B=37, N=64)
    _say(wl.name)
    data = I.generate(wl)
    gp = GpuProblem(wl, data)
    _, U_ref, hist_ref, _ = gp.forward()
    side = torch.cuda.Stream()                      # default priority
    gp.U.zero_()
    torch.cuda.synchronize()
    busy = torch.randn(2048, 2048, device="cuda")
    with torch.cuda.stream(side):
        rc, hist, it = M.mgrit_fas_forward(gp.p, gp.W, gp.b, gp.u0, gp.U, gp.ws, stream=side)
    for _ in range(4):
        busy = busy @ busy * 1e-3                   # default stream stays busy meanwhile
    side.synchronize()
    torch.cuda.synchronize()
    same = bool(np.array_equal(gp.U.cpu().numpy(), U_ref))
    assert same and hist == hist_ref


@pytest.mark.parametrize("layer", ["dense", "conv"])
def test_solves_recorded_into_a_hip_graph_replay_bitwise(layer):
    """A forward + adjoint pair without host outputs is kernel launches only: captured into a HIP graph it
    replays, several times and with eager work and synchronisations in between, to bitwise the eager result."""
    import torch
    import paper_2007_07336_amd as M
    if layer == "dense":
        wl = I.reduced(I.cfg2(2), name="dense_fp32_graph", q=136, B=70, N=64)
    else:
        wl = I.reduced(I.cfg3(2), name="conv_fp32_graph", C=16, Himg=12, Wimg=12, B=5, N=32)
    _say(wl.name)
    data = I.generate(wl)
    gp = GpuProblem(wl, data)
    lamN = torch.from_numpy(np.random.default_rng(3).standard_normal(wl.state_shape).astype(np.float32)).cuda()
    Lam = torch.zeros_like(gp.U)
    dW = torch.zeros(gp.W.shape, dtype=torch.float32, device="cuda")
    db = torch.zeros_like(gp.b)
    ws = torch.empty(M.mgrit_adjoint_workspace_bytes(gp.p), dtype=torch.uint8, device="cuda")

    def pair():
        M.mgrit_fas_forward(gp.p, gp.W, gp.b, gp.u0, gp.U, ws, want_hist=False)
        M.mgrit_fas_adjoint(gp.p, gp.W, gp.b, gp.U, lamN, Lam, dW, db, ws, want_hist=False)

    pair()
    torch.cuda.synchronize()
    ref = [t.clone() for t in (gp.U, Lam, dW, db)]
    side = torch.cuda.Stream()                      # default priority
    side.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(side):
        with torch.cuda.graph(graph, stream=side):
            pair()
    torch.cuda.synchronize()
    for replay in range(3):
        for t in (gp.U, Lam, dW, db):
            t.fill_(float(replay + 1))              # eager work between the replays
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        for t, r in zip((gp.U, Lam, dW, db), ref):
            assert torch.equal(t, r), replay


@pytest.mark.parametrize("layer", ["dense", "conv"])
def test_gradient_descent_with_early_stopped_multigrid(layer):
    """Loss goes down under gradient descent with two-cycle multigrid gradients and follows the loss curve of
    exact (serial) gradients; the first multigrid gradient is checked against the oracle's exact gradient."""
    import torch
    import paper_2007_07336_amd as M
    if layer == "dense":
        wl = I.reduced(I.cfg5(2), name="train_dense_fp32_q64_B32_N64", q=64, B=32, N=64, m=4, max_levels=3,
                       min_coarse=1, dtype=I.FP32, head_classes=10)
    else:
        wl = I.reduced(I.cfg3(2), name="train_conv_fp32_c8_8x8_B8_N32", B=8, C=8, Himg=8, Wimg=8, N=32, m=4,
                       max_levels=2, act=I.TANH, lifted_input=False, head_classes=10)
    _say(wl.name)
    data = I.generate(wl)
    dev = "cuda"
    W_o = torch.from_numpy(data["W_o"]).to(dev)
    labels = torch.from_numpy(data["labels"]).to(dev)

    def head(uN):                                    # mean cross-entropy of a linear head and d loss / d u^N
        x = uN.reshape(wl.B, -1).detach().requires_grad_(True)
        loss = torch.nn.functional.cross_entropy(x @ W_o.T, labels)
        (g,) = torch.autograd.grad(loss, x)
        return float(loss.detach()), g.reshape(uN.shape).contiguous()

    def run(levels, steps, lr):
        gp = GpuProblem(wl, data, max_levels=levels)
        nb = M.mgrit_adjoint_workspace_bytes(gp.p)
        ws = torch.empty(nb, dtype=torch.uint8, device=dev)
        Lam = torch.zeros_like(gp.U)
        dW = torch.zeros_like(gp.W)
        db = torch.zeros_like(gp.b)
        losses, first = [], None
        for _ in range(steps):
            M.mgrit_fas_forward(gp.p, gp.W, gp.b, gp.u0, gp.U, ws, want_hist=False)
            loss, lamN = head(gp.U[-1])
            M.mgrit_fas_adjoint(gp.p, gp.W, gp.b, gp.U, lamN, Lam, dW, db, ws, want_hist=False)
            if first is None:
                first = (dW.cpu().numpy().copy(), db.cpu().numpy().copy(), lamN.cpu().numpy().copy())
            gp.W -= lr * dW
            gp.b -= lr * db
            losses.append(loss)
        return losses, first

    lr = 20.0 if layer == "dense" else 5.0
    mg, first_mg = run(wl.max_levels, 15, lr)
    ser, first_ser = run(1, 15, lr)
    print("multigrid (2 cycles):", ["%.4f" % v for v in mg], "\nserial:              ", ["%.4f" % v for v in ser], flush=True)
    assert mg[-1] < 0.9 * mg[0] and ser[-1] < 0.9 * ser[0]
    assert all(b <= a + 1e-3 for a, b in zip(mg, mg[1:]))
    assert abs(mg[-1] - ser[-1]) <= 0.1 * (ser[0] - ser[-1])
    # the serial gradient of the first step against the oracle's exact backpropagation
    Us = O.serial_forward(data["W"], data["b"], data["u0"], wl.h, wl.layer, wl.act)
    _, dWo, dbo = O.serial_backward(data["W"], data["b"], Us, first_ser[2], wl.h, wl.layer, wl.act)
    assert rel_l2_per_state(first_ser[0], dWo) <= 1e-5 and rel_l2_per_state(first_ser[1], dbo) <= 1e-5
    # and the two-cycle multigrid gradient is close to it (Sec. IV-A: two cycles suffice)
    eW = float(np.linalg.norm(first_mg[0] - dWo) / np.linalg.norm(dWo))
    print(f"two-cycle gradient vs exact: {eW:.3e}", flush=True)
    assert eW <= 1e-2


@pytest.mark.parametrize("N", [64, 79])
@pytest.mark.parametrize("relax,levels,cycles", [(I.RELAX_F, 2, 1), (I.RELAX_FCF, 3, 2), (I.RELAX_FCF, 2, 3)])
def test_layer_step_count_of_the_benchmark_matches_the_launch_schedule(relax, levels, cycles, N):
    """bench.py's throughput numerator (layer steps per solve, from a closed formula) equals what the library
    actually launches: the launch trace counts one unit per group of every step launch."""
    import paper_2007_07336_amd as M
    import bench
    wl = I.reduced(I.cfg2(cycles), name="dense_fp32_step_count", q=64, B=8, N=N, m=4, max_levels=levels, relax=relax)
    _say(f"{wl.name} relax={relax} levels={levels} cycles={cycles}")
    data = I.generate(wl)
    gp = GpuProblem(wl, data)
    sizes, _ = M.mgrit_level_map(gp.p)
    M.mgrit_trace_begin()
    gp.forward()
    tr = M.mgrit_trace_end()
    units = sum(v[2] for k, v in tr.items() if k != "dense_grad_kernel")
    assert units == bench.layer_steps_per_solve(sizes, wl.m, wl.relax, cycles), (tr, sizes)


@pytest.mark.parametrize("sweep", [True, False], ids=["sweep", "lockstep"])
@pytest.mark.parametrize("relax", [I.RELAX_F, I.RELAX_FCF], ids=["F", "FCF"])
@pytest.mark.parametrize("row", [0, 1, 4, 9])
def test_known_value_inside_the_result_array(row, relax, sweep, monkeypatch):
    """u0 (lamN) may be a row of U (Lam), as where one solve continues from the last state of another in the same array: a
    C-point, an F-point or a trailing F-point, which the first relaxation writes to."""
    import torch
    import paper_2007_07336_amd as M
    if not sweep:
        monkeypatch.setenv("MGRIT_NO_SWEEP", "1")
    wl = I.reduced(I.cfg5(2), name="alias", q=64, B=16, N=9, m=4, max_levels=2, min_coarse=1, dtype=I.FP32, relax=relax, head_classes=0)
    _say(f"row {row} relax {relax} sweep {sweep}")
    gp = GpuProblem(wl, I.generate(wl))
    _, U, hist, _ = gp.forward()
    gp.U.fill_(7.0)
    gp.U[row] = gp.u0
    _, hist2, _ = M.mgrit_fas_forward(gp.p, gp.W, gp.b, gp.U[row], gp.U, gp.ws)
    assert np.array_equal(gp.U.cpu().numpy(), U) and hist2 == hist
    lamN = np.random.default_rng(2).standard_normal(wl.state_shape).astype(np.float32)
    Lam, _, _, hist, _ = gp.adjoint(U, lamN)
    Lam2 = torch.full_like(gp.U, 7.0)
    Lam2[row] = torch.from_numpy(lamN).cuda()
    ws = torch.empty(M.mgrit_adjoint_workspace_bytes(gp.p), dtype=torch.uint8, device="cuda")
    _, hist2, _ = M.mgrit_fas_adjoint(gp.p, gp.W, gp.b, gp.U, Lam2[row], Lam2, None, None, ws)
    assert np.array_equal(Lam2.cpu().numpy(), Lam) and hist2 == hist
