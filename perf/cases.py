"""Performance cases of the layer-parallel multigrid (MGRIT-FAS) library: whole forward and adjoint solves through
the public entry points, from the smallest stack (launches and latency) to the largest (memory and matrix cores).

A case is a dict: `kind` (dense, conv, or mixed = a convolution stack with periodic fully connected layers),
`pass` (forward, or adjoint = adjoint solve with the parameter gradient about given states), `dtype` (f32 or bf16 weights
and matrix operands), `act`, the hierarchy (`N`, `m`, `levels`, `min_coarse`, `fcf`, `cycles`), the sizes (`B` and `q`, or
`B`, `C`, `H`, `W`, and `period` of the fully connected layers) and `hist` (whether the caller asks for the residual
history, which makes the call wait for the GPU).
"""
import math
import random

import torch

import paper_2007_07336_amd as mgrit

DEV = "cuda" if torch.cuda.is_available() else "cpu"
RELU, TANH = "relu", "tanh"


def _dense(name, dtype, direction, q, B, N, m, levels, **kw):
    c = dict(kind="dense", dtype=dtype, q=q, B=B, N=N, m=m, levels=levels, min_coarse=1, fcf=True, cycles=2, act=RELU, hist=False)
    c.update(kw)
    c["name"], c["pass"] = name, direction
    return c


def _conv(name, dtype, direction, C, H, W, B, N, m, levels, **kw):
    c = dict(kind="conv", dtype=dtype, C=C, H=H, W=W, B=B, N=N, m=m, levels=levels, min_coarse=1, fcf=True, cycles=2, act=RELU,
             hist=False)
    c.update(kw)
    c["name"], c["pass"] = name, direction
    return c


def listed():
    return [
        # the smallest stack of the benchmark definitions (8 wide, 16 layers, batch 4, two levels, F-relaxation, four
        # cycles), called with the residual history: launch latency and the host path
        _dense("dense8_f32_forward", "f32", "forward", 8, 4, 16, 4, 2, fcf=False, cycles=4, act=TANH, hist=True),
        # a stack whose batch, width and depth are no multiples of any tile or of the coarsening factor
        _dense("dense200_f32_ragged_forward", "f32", "forward", 200, 50, 79, 4, 3, act=TANH, hist=True),
        # the benchmark's headline workload: width 256, 256 layers, batch 128, three levels, float: forward solve ...
        _dense("dense256_f32_forward", "f32", "forward", 256, 128, 256, 4, 3),
        # ... and the backward half of its training step: adjoint solve and parameter gradient
        _dense("dense256_f32_adjoint", "f32", "adjoint", 256, 128, 256, 4, 3),
        # the benchmark's small image stack: 16 channels, 28 x 28, 64 layers, batch 64, float
        _conv("conv16_f32_forward", "f32", "forward", 16, 28, 28, 64, 64, 4, 2),
        _conv("conv16_f32_adjoint", "f32", "adjoint", 16, 28, 28, 64, 64, 4, 2),
        # an odd image stack with a channel count between the compiled ones, deep in levels, F-relaxation, bf16
        _conv("conv24_bf16_odd_adjoint", "bf16", "adjoint", 24, 13, 17, 5, 45, 3, 3, fcf=False, act=TANH),
        # the benchmark's large image stack: 64 channels, 32 x 32, 512 layers, batch 32, bf16 operands
        _conv("conv64_bf16_forward", "bf16", "forward", 64, 32, 32, 32, 512, 8, 3),
        _conv("conv64_bf16_adjoint", "bf16", "adjoint", 64, 32, 32, 32, 512, 8, 3),
        # the benchmark's wide training stack: width 1024, 1024 layers, batch 256, bf16 operands
        _dense("dense1024_bf16_forward", "bf16", "forward", 1024, 256, 1024, 16, 8, min_coarse=8, act=TANH),
        _dense("dense1024_bf16_adjoint", "bf16", "adjoint", 1024, 256, 1024, 16, 8, min_coarse=8, act=TANH),
        # blocks of one fully connected layer (4096 wide, flattened images) and 63 convolution layers, float
        _conv("mixed16_f32_forward", "f32", "forward", 16, 16, 16, 32, 256, 4, 3, kind="mixed", period=64),
    ]


# --------------------------------------------------------------------------------------------- sizes and counts
def _sizes(c):
    """Steps of every level."""
    n = [c["N"]]
    while len(n) < c["levels"] and n[-1] > c["min_coarse"] and n[-1] >= c["m"]:
        n.append(n[-1] // c["m"])
    return n


def _steps(c):
    """Layer steps of one solve: relaxation, residual, coarse right-hand side and coarse solve of every cycle (the fine
    level's opening F-relaxation belongs to the first cycle only: it repeats the one that closed the cycle before)."""
    n, m = _sizes(c), c["m"]

    def f(l):
        return n[l] - n[l + 1]

    def cyc(l, first):
        if l == len(n) - 1:
            return n[l]
        s = (f(l) if first else 0) + (n[l + 1] + f(l) if c["fcf"] else 0) + 2 * n[l + 1] + cyc(l + 1, True) + f(l)
        return s

    if len(n) == 1:
        return c["N"]
    return sum(cyc(0, k == 0) for k in range(c["cycles"]))


def _geom(c):
    """(elements of a state, weights of a layer, multiply-adds of a layer step)."""
    if c["kind"] == "dense":
        return c["B"] * c["q"], c["q"] ** 2, c["B"] * c["q"] ** 2
    M = c["B"] * c["H"] * c["W"]
    return M * c["C"], 9 * c["C"] ** 2, M * 9 * c["C"] ** 2


def _fc(c):
    """(number of fully connected layers, flattened sample size)."""
    if c["kind"] != "mixed":
        return 0, 0
    return -(-c["N"] // c["period"]), c["H"] * c["W"] * c["C"]


def work(case):
    c = case
    E, ws, macs = _geom(c)
    nfc, d = _fc(c)
    eb = 4 if c["dtype"] == "f32" else 2
    nw = c["N"] - nfc
    weights = nw * ws + nfc * d * d
    # a step of a mixed stack, averaged over its two kinds of layer
    macs = (nw * macs + nfc * c["B"] * d * d) / c["N"]
    bias = 4 * (nw * (c["q"] if c["kind"] == "dense" else c["C"]) + nfc * d)
    states = 4 * E * (c["N"] + 1)
    flops = 2.0 * macs * _steps(c)
    b = eb * weights + bias + 4 * E + states                      # parameters and the known value in, all states out
    if c["pass"] == "adjoint":
        b += states + 4 * weights + bias                          # states to linearise about in, gradients out
        flops += 4.0 * macs * c["N"]                              # act' of every layer and the parameter gradient
    return {"bytes": float(b), "flops": flops}


# --------------------------------------------------------------------------------------------- drawn cases
_LARGEST = 9.0e12          # multiply-adds count twice: just below the largest listed case


def draw(rng: random.Random):
    def logint(lo, hi, mult=1):
        return max(1, round(math.exp(rng.uniform(math.log(lo), math.log(hi))) / mult)) * mult

    while True:
        kind = rng.choice(["dense", "dense", "dense", "conv", "conv", "conv", "mixed"])
        c = dict(kind=kind, dtype=rng.choice(["f32", "bf16"]), m=rng.choice([2, 3, 4, 4, 5, 8, 8, 16]), levels=rng.randint(2, 4),
                 min_coarse=rng.choice([1, 1, 4, 8]), fcf=rng.random() < 0.7, cycles=rng.randint(1, 3), act=rng.choice([RELU, TANH]),
                 hist=rng.random() < 0.3)
        c["pass"] = rng.choice(["forward", "adjoint"])
        if kind == "dense":
            c.update(q=logint(8, 1024, 8), B=logint(2, 256), N=logint(16, 1024))
            if rng.random() < 0.4:                               # widths and batches of the usual kind among the odd ones
                c.update(q=rng.choice([64, 128, 256, 512, 1024]), B=rng.choice([16, 32, 64, 128, 256]))
        elif kind == "conv":
            c.update(C=rng.choice([8, 16, 16, 24, 32, 48, 64, 64]), H=rng.randint(5, 32), W=rng.randint(5, 32), B=logint(2, 64),
                     N=logint(16, 512))
            if rng.random() < 0.4:
                c["H"] = c["W"] = rng.choice([8, 14, 16, 28, 32])
        else:
            c.update(C=rng.choice([8, 16]), H=rng.randint(5, 16), W=rng.randint(5, 16), B=logint(4, 32), N=logint(16, 256),
                     period=rng.randint(4, 64))
        if c["N"] < 2 * c["m"]:
            continue
        E, ws, _ = _geom(c)
        nfc, d = _fc(c)
        small = 16 * E * (c["N"] + 1) < 2.0e10 and 8 * (c["N"] * ws + nfc * d * d) < 1.2e10   # fits, and is quickly made
        if small and work(c)["flops"] <= _LARGEST:
            return c


# --------------------------------------------------------------------------------------------- inputs
def _grid(x, step):
    return torch.round(x / step) * step


def _inputs(c, seed):
    """Random layers and samples of the benchmark's distributions (float32 values; weights of a bf16 case are
    representable in bf16): W ~ N(0, 1/q) or N(0, 2/(9 C)), b ~ N(0, 0.1), u0 ~ N(0, 1), and for the adjoint the terminal
    value and the states of serial propagation.

    ReLU' is a 0/1 decision that the order of a sum can turn where a pre-activation is nearly zero, and one turned decision
    is worth more than all rounding.  So a ReLU stack is linearised about states (and with float weights and biases) on binary
    grids on which the pre-activations are exact in any order, and bf16 stacks about states that bf16 represents."""
    g = torch.Generator(device=DEV).manual_seed(seed)

    def normal(shape, var):
        return torch.randn(shape, generator=g, device=DEV, dtype=torch.float32) * math.sqrt(var)

    x = {}
    exact_z = c["pass"] == "adjoint" and c["act"] == RELU
    nfc, d = _fc(c)
    if c["kind"] == "dense":
        var, shape, feat = 1.0 / c["q"], (c["N"], c["q"], c["q"]), c["q"]
        x["u0"] = normal((c["B"], c["q"]), 1.0)
    else:
        var, shape, feat = 2.0 / (9 * c["C"]), (c["N"], c["C"], 3, 3, c["C"]), c["C"]
        x["u0"] = normal((c["B"], c["H"], c["W"], c["C"]), 1.0)
    x["W"] = normal(shape, var)
    x["b"] = normal((c["N"], feat), 0.1)
    if nfc:
        x["Wfc"] = normal((nfc, d, d), 1.0 / d)
        x["bfc"] = normal((nfc, d), 0.1)
    for k in ("W", "Wfc"):
        if k in x:
            if exact_z:                                      # six significant bits below the spread of the weights
                s = math.sqrt(var if k == "W" else 1.0 / d)
                x[k] = _grid(x[k], 2.0 ** (math.floor(math.log2(s)) - 4))
            if c["dtype"] == "bf16":
                x[k] = x[k].to(torch.bfloat16)
    if exact_z:
        for k in ("b", "bfc"):
            if k in x:
                x[k] = _grid(x[k], 2.0 ** -10)
    if c["pass"] == "adjoint":
        U = torch.empty((c["N"] + 1,) + tuple(x["u0"].shape), device=DEV, dtype=torch.float32)
        u = x["u0"].clone()
        for n in range(c["N"] + 1):
            U[n] = _grid(u, 2.0 ** -5) if exact_z else u.to(torch.bfloat16).float() if c["dtype"] == "bf16" else u
            if n < c["N"]:
                u = u + _act(_affine(c, x, u[None], [n], torch.float32), c["act"])[0] / c["N"]
        x["U"] = U
        x["lamN"] = normal(tuple(x["u0"].shape), 1.0) / c["B"]
    return x


def prepare(case, seed):
    c = case
    x = _inputs(c, seed)
    p = mgrit.make_problem(N=c["N"], h=1.0 / c["N"], m=c["m"], max_levels=c["levels"], min_coarse=c["min_coarse"],
                           relax=1 if c["fcf"] else 0, max_iter=c["cycles"], layer=0 if c["kind"] == "dense" else 1,
                           act=1 if c["act"] == RELU else 0, dtype=0 if c["dtype"] == "f32" else 1, B=c["B"], q=c.get("q", 0),
                           C=c.get("C", 0), Himg=c.get("H", 0), Wimg=c.get("W", 0))
    s = dict(x, p=p, hist=c["hist"], adjoint=c["pass"] == "adjoint")
    new = lambda t: torch.empty(t.shape, device=DEV, dtype=torch.float32)                      # noqa: E731
    if c["kind"] == "mixed":
        if s["adjoint"]:
            s["dWfc"], s["dbfc"] = new(x["Wfc"]), new(x["bfc"])
        s["fc"] = mgrit.make_fc_layers(c["period"], x["Wfc"], x["bfc"], s.get("dWfc"), s.get("dbfc"))
        need = mgrit.mgrit_adjoint_workspace_bytes_mixed if s["adjoint"] else mgrit.mgrit_workspace_bytes_mixed
        nbytes = need(p, c["period"])
    else:
        need = mgrit.mgrit_adjoint_workspace_bytes if s["adjoint"] else mgrit.mgrit_workspace_bytes
        nbytes = need(p)
    s["ws"] = torch.empty(nbytes, device=DEV, dtype=torch.uint8)
    if s["adjoint"]:
        s["Lam"], s["dW"], s["db"] = new(x["U"]), new(x["W"]), new(x["b"])
    else:
        s["U"] = torch.empty((c["N"] + 1,) + tuple(x["u0"].shape), device=DEV, dtype=torch.float32)
    return s


def run(state):
    s = state
    if not s["adjoint"]:
        if "fc" in s:
            mgrit.mgrit_fas_forward_mixed(s["p"], s["fc"], s["W"], s["b"], s["u0"], s["U"], s["ws"], want_hist=s["hist"])
        else:
            mgrit.mgrit_fas_forward(s["p"], s["W"], s["b"], s["u0"], s["U"], s["ws"], want_hist=s["hist"])
        return {"U": s["U"]}
    if "fc" in s:
        mgrit.mgrit_fas_adjoint_mixed(s["p"], s["fc"], s["W"], s["b"], s["U"], s["lamN"], s["Lam"], s["dW"], s["db"], s["ws"],
                                      want_hist=s["hist"])
        return {"Lam": s["Lam"], "dW": s["dW"], "db": s["db"], "dWfc": s["dWfc"], "dbfc": s["dbfc"]}
    mgrit.mgrit_fas_adjoint(s["p"], s["W"], s["b"], s["U"], s["lamN"], s["Lam"], s["dW"], s["db"], s["ws"], want_hist=s["hist"])
    return {"Lam": s["Lam"], "dW": s["dW"], "db": s["db"]}


def tolerance(case):
    # float: sums of up to 9 C or q terms in another order, carried through the cycle; bf16: the operands are rounded to
    # bf16 from float states that differ in their last bits, and the gradient's operands likewise
    if case["dtype"] == "f32":
        return {"rel": 5e-6, "max": 5e-4}
    return {"rel": 4e-3, "max": 2e-1}


# --------------------------------------------------------------------------------------------- the same in 64 bits
def _act(z, act):
    return torch.relu(z) if act == RELU else torch.tanh(z)


def _is_fc(c, n):
    return c["kind"] == "mixed" and n % c["period"] == 0


def _taps(u, flip=1):
    """The nine shifted copies of images u [..., H, W, C] with one pixel of zeros around them: ((dy, dx), copy)."""
    p = torch.nn.functional.pad(u, (0, 0, 1, 1, 1, 1))
    H, W = u.shape[-3], u.shape[-2]
    for dy in range(3):
        for dx in range(3):
            oy, ox = (dy, dx) if flip == 1 else (2 - dy, 2 - dx)
            yield dy, dx, p[..., oy:oy + H, ox:ox + W, :]


def _affine(c, x, u, layers, dt):
    """A u + b of group g's layer layers[g] on u[g]."""
    z = torch.empty_like(u)
    conv = [g for g, n in enumerate(layers) if not _is_fc(c, n)]
    if conv:
        n = [layers[g] for g in conv]
        W, b = x["W"][n].to(dt), x["b"][n].to(dt)
        v = u if len(conv) == len(layers) else u[conv]
        if c["kind"] == "dense":
            r = torch.matmul(v, W.transpose(1, 2).contiguous()) + b[:, None]
        else:
            r = b[:, None, None, None, :].expand(v.shape).reshape(len(n), -1, c["C"]).clone()
            for dy, dx, t in _taps(v):
                r += torch.matmul(t.reshape(len(n), -1, c["C"]), W[:, :, dy, dx, :].transpose(1, 2).contiguous())
            r = r.reshape(v.shape)
        z[conv] = r
    for g, n in enumerate(layers):
        if _is_fc(c, n):
            k = n // c["period"]
            z[g] = (u[g].reshape(c["B"], -1) @ x["Wfc"][k].to(dt).T + x["bfc"][k].to(dt)).reshape(u[g].shape)
    return z


def _affine_t(c, x, G, layers):
    """A^T G of group g's layer (64 bits)."""
    r = torch.empty_like(G)
    conv = [g for g, n in enumerate(layers) if not _is_fc(c, n)]
    if conv:
        n = [layers[g] for g in conv]
        W = x["W"][n].double()
        v = G if len(conv) == len(layers) else G[conv]
        if c["kind"] == "dense":
            r[conv] = torch.matmul(v, W.contiguous())
        else:
            s = torch.zeros_like(v).reshape(len(n), -1, c["C"])
            for dy, dx, t in _taps(v, flip=-1):
                s += torch.matmul(t.reshape(len(n), -1, c["C"]), W[:, :, dy, dx, :].contiguous())
            r[conv] = s.reshape(v.shape)
    for g, n in enumerate(layers):
        if _is_fc(c, n):
            k = n // c["period"]
            r[g] = (G[g].reshape(c["B"], -1) @ x["Wfc"][k].double()).reshape(G[g].shape)
    return r


def _solve(c, first, step):
    """The FAS cycles on sweep points 0..N from the known value `first`, C-points started at it; step(l, j, v) advances states
    v[g] of level l from point j[g] - 1 to point j[g]."""
    n, m = _sizes(c), c["m"]
    X = [torch.zeros((k + 1,) + tuple(first.shape), device=first.device, dtype=torch.float64) for k in n]
    rhs = [None] * len(n)
    CH = max(1, int(4.0e9 / (8 * first.numel())))                     # groups advanced at once, by memory

    def put(l, js):
        for a in range(0, len(js), CH):
            j = js[a:a + CH]
            v = step(l, j, X[l][[i - 1 for i in j]])
            X[l][j] = v if rhs[l] is None else v + rhs[l][j]

    def f_relax(l):
        for k in range(1, m):
            js = list(range(k, n[l] + 1, m))
            if js:
                put(l, js)

    def cycle(l):
        if l == len(n) - 1:
            for j in range(1, n[l] + 1):
                put(l, [j])
            return
        C = list(range(m, n[l + 1] * m + 1, m))
        f_relax(l)
        if c["fcf"]:
            put(l, C)
            f_relax(l)
        # coarse equation L_H(V) = L_H(U_H) + R_H with V started at the injected states
        X[l + 1] = X[l][::m][:n[l + 1] + 1].clone()
        rhs[l + 1] = torch.zeros_like(X[l + 1])
        rhs[l + 1][0] = first
        for a in range(0, len(C), CH):
            j = C[a:a + CH]
            J = [i // m for i in j]
            R = step(l, j, X[l][[i - 1 for i in j]]) - X[l][j]
            if rhs[l] is not None:
                R += rhs[l][j]
            rhs[l + 1][J] = X[l + 1][J] - step(l + 1, J, X[l + 1][[i - 1 for i in J]]) + R
        cycle(l + 1)
        X[l][C] = X[l + 1][1:]
        f_relax(l)

    X[0][0] = first
    if len(n) == 1:
        cycle(0)
        return X[0]
    X[0][m::m] = first
    for _ in range(c["cycles"]):
        cycle(0)
    return X[0]


def exact(case, seed):
    c, m, N = case, case["m"], case["N"]
    x = _inputs(c, seed)
    h = 1.0 / N
    if c["pass"] == "forward":
        def step(l, js, v):
            return v + h * m ** l * _act(_affine(c, x, v, [(j - 1) * m ** l for j in js], torch.float64), c["act"])
        return {"U": _solve(c, x["u0"].double(), step)}

    E = x["u0"].numel()
    D = torch.empty((N,) + tuple(x["u0"].shape), device=DEV, dtype=torch.float64)
    CH = max(1, int(4.0e9 / (8 * E)))
    for a in range(0, N, CH):
        ns = list(range(a, min(N, a + CH)))
        z = _affine(c, x, x["U"][ns].double(), ns, torch.float64)
        D[ns] = (z > 0).double() if c["act"] == RELU else 1.0 - torch.tanh(z) ** 2

    def back(l, js, v):                            # sweep point j of level l is layer point N - j m^l
        ns = [N - j * m ** l for j in js]
        return v + h * m ** l * _affine_t(c, x, D[ns] * v, ns)
    Lam = _solve(c, x["lamN"].double(), back).flip(0)
    out = {"Lam": Lam, "dW": torch.zeros(x["W"].shape, device=DEV, dtype=torch.float64),
           "db": torch.zeros(x["b"].shape, device=DEV, dtype=torch.float64)}
    if c["kind"] == "mixed":
        out["dWfc"] = torch.zeros(x["Wfc"].shape, device=DEV, dtype=torch.float64)
        out["dbfc"] = torch.zeros(x["bfc"].shape, device=DEV, dtype=torch.float64)
    for n in range(N):
        G, u = h * D[n] * Lam[n + 1], x["U"][n].double()
        if c["kind"] == "dense" or _is_fc(c, n):
            k, w, b = (n, "dW", "db") if c["kind"] == "dense" else (n // c["period"], "dWfc", "dbfc")
            G, u = G.reshape(c["B"], -1), u.reshape(c["B"], -1)
            out[w][k] = G.T.contiguous() @ u
            out[b][k] = G.sum(0)
            continue
        Gt = G.reshape(-1, c["C"]).T.contiguous()
        for dy, dx, t in _taps(u):
            out["dW"][n, :, dy, dx, :] = Gt @ t.reshape(-1, c["C"])
        out["db"][n] = G.reshape(-1, c["C"]).sum(0)
    return out
