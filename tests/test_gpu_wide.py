"""Sweep over dense bf16 layers of width 257 to 1024: slices of 64 rows that are not full, widths that end inside a pass, a block or
a k step, trailing F-points, both directions, both storages of the act' factors; up to width 520 against the CPU oracle, above
against the lockstep launches (MGRIT_NO_SWEEP=1), which the other tests hold against it.  Tolerance 2e-2 (relative L2), that of bf16
operands; between the two kernels, which round the same operands and differ in the order of float sums, 1e-3, and 1e-2 for the
gradient, whose operands may round the other way."""
import numpy as np
import pytest

import mgrit_inputs as I
from tests.gpu_util import GpuProblem, oracle_forward, oracle_adjoint, rel_l2_per_state

pytestmark = pytest.mark.gpu


def _dense(q, B, N, m, levels=2, relax=I.RELAX_FCF, act=I.TANH, it=2):
    return I.reduced(I.cfg5(it), name=f"wide_q{q}_B{B}_N{N}_m{m}_{'FCF' if relax else 'F'}_{'relu' if act else 'tanh'}", q=q, B=B, N=N, m=m,
                     max_levels=levels, min_coarse=1, relax=relax, act=act, head_classes=0)


ORACLE = [_dense(264, 5, 146, 2), _dense(320, 1, 147, 2, act=I.RELU, relax=I.RELAX_F), _dense(392, 70, 80, 2, levels=3), _dense(512, 64, 147, 2),
          _dense(520, 130, 66, 2, relax=I.RELAX_F)]


@pytest.mark.parametrize("wl", ORACLE, ids=[w.name for w in ORACLE])
def test_against_the_oracle(wl):
    print(f"\n[case] {wl.name}", flush=True)
    data = I.generate(wl)
    gp = GpuProblem(wl, data)
    gp.M.mgrit_trace_begin()
    _, U, hist, it = gp.forward()
    tr = gp.M.mgrit_trace_end()
    assert any("sweep" in k for k in tr), tr
    Uo, hist_o, it_o = oracle_forward(wl, data)
    assert it == it_o and rel_l2_per_state(U, Uo) <= 2e-2
    assert all(abs(a - b) <= 0.2 * b + 1e-4 for a, b in zip(hist, hist_o)), (hist, hist_o)
    if wl.act == I.RELU:
        return                                   # ReLU' is a 0/1 decision that the operands' rounding can turn
    lamN = np.random.default_rng(1).standard_normal(wl.state_shape).astype(np.float32)
    Lam, dW, db, _, _ = gp.adjoint(U, lamN)
    Lo, dWo, dbo, _, _ = oracle_adjoint(wl, data, U.astype(np.float64), lamN)
    assert rel_l2_per_state(Lam, Lo) <= 2e-2
    assert np.linalg.norm(dW - dWo) <= 2e-2 * np.linalg.norm(dWo) and np.linalg.norm(db - dbo) <= 2e-2 * np.linalg.norm(dbo)


@pytest.mark.parametrize("transposed", [False, True], ids=["as_stored", "transposed"])
@pytest.mark.parametrize("q,B,N,m,relu", [(640, 100, 96, 2, False), (768, 65, 150, 2, True), (776, 193, 82, 2, False), (1000, 3, 330, 2, True), (1024, 256, 81, 2, False)])
def test_against_lockstep_launches(q, B, N, m, relu, transposed, monkeypatch):
    import torch
    import paper_2007_07336_amd as M
    print(f"\n[case] q{q} B{B} N{N}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(q)
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda")                                     # noqa: E731
    p = M.make_problem(N=N, h=1.0 / N, m=m, max_levels=2, min_coarse=1, relax=1, max_iter=1, layer=0, act=1 if relu else 0, dtype=1, B=B, q=q)
    W, b = (rnd(N, q, q) / q ** 0.5).bfloat16(), 0.3 * rnd(N, q)
    if transposed:
        monkeypatch.setenv("MGRIT_ADJ_TRANSPOSED", "1")
    ws = torch.empty(M.mgrit_adjoint_workspace_bytes(p), dtype=torch.uint8, device="cuda")
    Uin, lam, res = rnd(N + 1, B, q).bfloat16().float(), rnd(B, q), []
    for off in (False, True):
        if off:
            monkeypatch.setenv("MGRIT_NO_SWEEP", "1")
        U, Lam, dW, db = torch.full_like(Uin, float("nan")), torch.full_like(Uin, float("nan")), torch.empty(N, q, q, device="cuda"), torch.empty_like(b)
        M.mgrit_trace_begin()
        M.mgrit_fas_forward(p, W, b, Uin[0], U, ws)
        M.mgrit_fas_adjoint(p, W, b, Uin, lam, Lam, dW, db, ws)
        torch.cuda.synchronize()
        tr = M.mgrit_trace_end()
        assert any("sweep" in k for k in tr) == (not off), tr
        res.append((U, Lam, dW, db))
    for x, y, tol in zip(res[0], res[1], (1e-3, 1e-3, 1e-2, 1e-3)):
        assert float((x - y).norm()) <= tol * float(y.norm())


def test_infinite_weights_past_the_width(monkeypatch):
    """The weights that a lane reads for values of k past the width, the next row's first, are infinite: the sweep ends with the same
    NaN as the lockstep launches, none in the first step's feature 0, whose own weights are zeros."""
    import torch
    import paper_2007_07336_amd as M
    q, B, N = 296, 40, 160
    p = M.make_problem(N=N, h=1.0 / N, m=2, max_levels=2, min_coarse=1, relax=0, max_iter=1, layer=0, act=0, dtype=1, B=B, q=q)
    W = torch.zeros(N, q, q, device="cuda", dtype=torch.bfloat16)
    W[:, 1:, :24] = float("inf")
    u0 = torch.zeros(B, q, device="cuda")
    u0[:, 24:] = 1.0
    res, ws = [], torch.empty(M.mgrit_workspace_bytes(p), dtype=torch.uint8, device="cuda")
    for off in (False, True):
        if off:
            monkeypatch.setenv("MGRIT_NO_SWEEP", "1")
        U = torch.empty(N + 1, B, q, device="cuda")
        M.mgrit_fas_forward(p, W, torch.zeros(N, q, device="cuda"), u0, U, ws, want_hist=False, check=False)
        torch.cuda.synchronize()
        res.append(U)
    assert bool((res[0][1, :, 0] == 0).all())
    assert torch.equal(res[0].isnan(), res[1].isnan()) and torch.equal(res[0].nan_to_num(), res[1].nan_to_num())


@pytest.mark.parametrize("q,m,N,relu", [(512, 2, 80, True), (640, 2, 100, False), (1000, 2, 100, False), (1024, 3, 150, True)])
def test_a_sample_ends_the_same_wherever_it_is_in_the_batch(q, m, N, relu):
    """Four slices of 64 rows with the same samples: the same states and multipliers, bit for bit, as in lockstep launches."""
    import torch
    import paper_2007_07336_amd as M
    g = torch.Generator(device="cuda").manual_seed(q)
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda")                                     # noqa: E731
    p = M.make_problem(N=N, h=1.0 / N, m=m, max_levels=2, min_coarse=1, relax=1, max_iter=1, layer=0, act=1 if relu else 0, dtype=1, B=256, q=q)
    W, b = (rnd(N, q, q) / q ** 0.5).bfloat16(), 0.3 * rnd(N, q)
    u0, lam = rnd(64, q).repeat(4, 1), rnd(64, q).repeat(4, 1)
    ws = torch.empty(M.mgrit_adjoint_workspace_bytes(p), dtype=torch.uint8, device="cuda")
    U, Lam = torch.empty(N + 1, 256, q, device="cuda"), torch.empty(N + 1, 256, q, device="cuda")
    M.mgrit_trace_begin()
    M.mgrit_fas_forward(p, W, b, u0, U, ws)
    M.mgrit_fas_adjoint(p, W, b, U, lam, Lam, None, None, ws)
    torch.cuda.synchronize()
    tr = M.mgrit_trace_end()
    assert any("sweep" in k for k in tr), tr
    for x in (U, Lam):
        for i in range(1, 4):
            assert not bool((x[:, 64 * i:64 * i + 64] != x[:, :64]).any())


# rows, chains: workgroups of 64 rows, 256 to a round
@pytest.mark.parametrize("q,B,chains,direction,sweep", [
    (776, 128, 79, "forward", False), (776, 128, 80, "forward", True), (776, 128, 128, "forward", True), (776, 128, 129, "forward", False),
    (776, 128, 199, "adjoint", False), (776, 128, 200, "adjoint", True), (776, 70, 299, "forward", False), (776, 70, 300, "forward", True),
    (776, 256, 193, "adjoint", True), (776, 64, 257, "forward", True), (904, 128, 99, "adjoint", False), (904, 128, 100, "adjoint", True),
    (904, 128, 99, "forward", True), (648, 128, 171, "forward", False), (648, 128, 172, "forward", True), (520, 128, 143, "adjoint", False),
    (520, 128, 144, "adjoint", True), (512, 128, 129, "forward", True)])
def test_kernel_choice_where_a_round_of_workgroups_begins(q, B, chains, direction, sweep, monkeypatch):
    """Which kernel relaxes the fine level, and that both give the same result there."""
    import torch
    import paper_2007_07336_amd as M
    print(f"\n[case] q{q} B{B} {chains} chains {direction}", flush=True)
    N = 2 * chains
    g = torch.Generator(device="cuda").manual_seed(q)
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda")                                     # noqa: E731
    p = M.make_problem(N=N, h=1.0 / N, m=2, max_levels=2, min_coarse=1, relax=0, max_iter=1, layer=0, act=0, dtype=1, B=B, q=q)
    W, b, U, first = (rnd(N, q, q) / q ** 0.5).bfloat16(), 0.3 * rnd(N, q), rnd(N + 1, B, q), rnd(B, q)
    ws, res = torch.empty(M.mgrit_adjoint_workspace_bytes(p), dtype=torch.uint8, device="cuda"), []
    for off in (False, True):
        if off:
            monkeypatch.setenv("MGRIT_NO_SWEEP", "1")
        X = torch.full_like(U, float("nan"))
        M.mgrit_trace_begin()
        if direction == "forward":
            M.mgrit_fas_forward(p, W, b, first, X, ws, want_hist=False)
        else:
            M.mgrit_fas_adjoint(p, W, b, U, first, X, None, None, ws, want_hist=False)
        torch.cuda.synchronize()
        assert any("sweep" in k for k in M.mgrit_trace_end()) == (sweep and not off)
        res.append(X)
    assert float((res[0] - res[1]).norm()) <= 1e-3 * float(res[1].norm())
