"""Performance cases: the work a user of the library has it do, through its
public entry points.

A case is a plain dict: a path (what is called), a problem with its grid, and
the options of the call.  `listed()` holds the named cases, `draw(rng)` makes
more of the same ranges, `prepare(case, seed)` makes the inputs on the GPU,
`run(state)` is one pass, `work(case)` what a pass cannot do without and
`exact(case, seed)` its results in 64 bits without the library.

Paths
  setup_solve  one hierarchy set up, one system solved, the hierarchy released
               (a steady-state run; the library's headline use)
  solve        a solve on a kept hierarchy (time steps with one operator)
  multi        a block solve of several right-hand sides on a kept hierarchy
  batch        independent systems set up and solved together
  resetup      new coefficients on a kept pattern, then a solve (Newton steps)
  train        one training step of the learned smoother weights
  spmv         the sparse product on a caller's CSR matrix (a residual check)
"""
import math

import numpy as np
import torch

import paper_1403_1649_amd as amg
from paper_1403_1649_amd import learned

RTOL = 1e-8

# outer iterations to 1e-8 with the default options (damped Jacobi, K-cycles on
# two levels), rounded: the method's own count, which no implementation avoids
ITERATIONS = {"poisson2d": 19, "aniso2d": 27, "poisson3d": 18, "aniso3d": 19, "hetero3d": 36, "convdiff2d": 19}


def listed():
    return [
        # the smallest call in use: a 2-D Poisson problem, where launches and read-backs are the time
        dict(name="poisson2d_128_fp64", path="setup_solve", problem="poisson2d", nx=128, ny=128, nz=1,
             precision="fp64"),
        # an ordinary 3-D Poisson solve, set-up included
        dict(name="poisson3d_128_fp64", path="setup_solve", problem="poisson3d", nx=128, ny=128, nz=128,
             precision="fp64"),
        # the largest: pressure equation with log-normal coefficients (reservoir simulation)
        dict(name="hetero3d_160_fp64", path="setup_solve", problem="hetero3d", nx=160, ny=160, nz=160,
             precision="fp64"),
        # the same operator kept over time steps, FP32 cycle inside FP64 flexible CG
        dict(name="hetero3d_160_mixed_solve", path="solve", problem="hetero3d", nx=160, ny=160, nz=160,
             precision="mixed"),
        # odd, ragged grid with the polynomial smoother, mixed precision
        dict(name="poisson3d_odd_cheb_mixed", path="setup_solve", problem="poisson3d", nx=113, ny=87, nz=61,
             precision="mixed", smoother="chebyshev"),
        # many right-hand sides (sources) against one anisotropic operator
        dict(name="aniso3d_96_rhs32_mixed", path="multi", problem="aniso3d", nx=96, ny=96, nz=96,
             precision="mixed", nrhs=32),
        # a few right-hand sides on a small odd grid, all in FP64
        dict(name="hetero3d_41_rhs5_fp64", path="multi", problem="hetero3d", nx=41, ny=43, nz=40,
             precision="fp64", nrhs=5),
        # 64 uneven 2-D systems in one batch
        dict(name="batch2d_64_mixed", path="batch", problem="poisson2d", nsys=64, lo=64, hi=512, layout=3,
             precision="mixed"),
        # a Newton step: new coefficients on the kept pattern, then the solve
        dict(name="hetero3d_96_resetup", path="resetup", problem="hetero3d", nx=96, ny=96, nz=96,
             precision="fp64"),
        # nonsymmetric convection-diffusion: flexible GMRES outside, the GMRES K-cycle inside
        dict(name="convdiff2d_500_fgmres", path="setup_solve", problem="convdiff2d", nx=500, ny=500, nz=1,
             precision="fp64", krylov="fgmres"),
        # one Adam step of the learned smoother weights on a training field, 8 error samples
        dict(name="hetero3d_64_train", path="train", problem="hetero3d", nx=64, ny=64, nz=64, samples=8,
             precision="fp64"),
        # the sparse product alone, on the caller's CSR arrays
        dict(name="hetero3d_160_spmv", path="spmv", problem="hetero3d", nx=160, ny=160, nz=160,
             precision="fp64"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    path = rng.choice(["setup_solve"] * 5 + ["solve", "solve", "multi", "multi", "batch", "resetup", "train", "spmv"])
    c = dict(path=path, precision=rng.choice(["fp64", "fp64", "mixed"]))
    if path == "batch":
        lo = _log_int(rng, 24, 128)
        c.update(problem="poisson2d", nsys=_log_int(rng, 2, 64), lo=lo, hi=lo + _log_int(rng, 8, 384),
                 layout=rng.randrange(1000))
        return c
    if path in ("train", "resetup"):
        c.update(problem="hetero3d", precision="fp64")
        side = _log_int(rng, 20, 72 if path == "train" else 110)
        if path == "train":
            c["samples"] = rng.choice([4, 8, 8, 16])
    elif path == "multi":
        c["problem"] = rng.choice(["poisson3d", "aniso3d", "hetero3d"])
        c["nrhs"] = _log_int(rng, 2, 33)
        side = _log_int(rng, 16, 72)
    elif path == "spmv":
        c.update(problem=rng.choice(["poisson3d", "hetero3d", "poisson2d"]), precision="fp64")
        side = _log_int(rng, 24, 159)
    else:
        c["problem"] = rng.choice(["poisson2d", "aniso2d", "poisson3d", "aniso3d", "hetero3d", "convdiff2d"])
        side = _log_int(rng, 16, 120)
        if c["problem"] == "convdiff2d":
            c["krylov"] = "fgmres"
        elif path == "setup_solve":
            c["smoother"] = rng.choice(["jacobi", "jacobi", "jacobi", "chebyshev"])
            c["kcycle_levels"] = rng.choice([2, 2, 2, 1])
            c["mis_k"] = rng.choice([2, 2, 2, 3])
    ratio = [rng.uniform(0.75, 1.3) for _ in range(3)]
    if c["problem"].endswith("2d"):
        side = int(round(side ** 1.4))   # 2-D grids of a comparable range: 48 to 816 a side
        if c["problem"] == "convdiff2d":
            side = min(side, 600)
        c.update(nx=max(12, int(side * ratio[0])), ny=max(12, int(side * ratio[1])), nz=1)
    else:
        c.update(nx=max(8, int(side * ratio[0])), ny=max(8, int(side * ratio[1])), nz=max(8, int(side * ratio[2])))
    return c


# ---------------------------------------------------------------- matrices
# Seven slots per row in ascending column order: z-, y-, x-, diagonal, x+, y+,
# z+ (x fastest); a boundary's slots are masked out.


def _faces(case, seed):
    """Coupling to the +1 neighbour along z, y, x (grid-shaped, the last plane
    unused) and the diagonal, float64 on the GPU."""
    shape = (case["nz"], case["ny"], case["nx"])
    one = torch.ones(shape, dtype=torch.float64, device="cuda")
    p = case["problem"]
    if p in ("poisson2d", "convdiff2d"):
        return [None, one, one], 4.0 * one
    if p == "aniso2d":
        return [None, 1e-3 * one, one], (2.0 + 2e-3) * one
    if p == "poisson3d":
        return [one, one, one], 6.0 * one
    if p == "aniso3d":
        return [1e-3 * one, one, one], (4.0 + 2e-3) * one
    # two-point-flux finite volumes, cell permeability exp(2 g), harmonic face
    # averages, Dirichlet x-faces, no flux through the others
    g = torch.Generator(device="cuda").manual_seed(int(seed))
    k = torch.exp(2.0 * torch.randn(shape, dtype=torch.float64, device="cuda", generator=g))
    diag = torch.zeros(shape, dtype=torch.float64, device="cuda")
    faces = []
    for ax in range(3):
        a, b = k.narrow(ax, 0, shape[ax] - 1), k.narrow(ax, 1, shape[ax] - 1)
        t = 2.0 * a * b / (a + b)
        diag.narrow(ax, 0, shape[ax] - 1).add_(t)
        diag.narrow(ax, 1, shape[ax] - 1).add_(t)
        full = torch.zeros(shape, dtype=torch.float64, device="cuda")
        full.narrow(ax, 0, shape[ax] - 1).copy_(t)
        faces.append(full)
    diag[:, :, 0] += 2.0 * k[:, :, 0]
    diag[:, :, -1] += 2.0 * k[:, :, -1]
    return faces, diag


def _slots(case, seed):
    """(columns [n,7] int64, values [n,7], mask [n,7]) of the matrix."""
    shape = (case["nz"], case["ny"], case["nx"])
    n = shape[0] * shape[1] * shape[2]
    faces, diag = _faces(case, seed)
    idx = torch.arange(n, device="cuda").reshape(shape)
    col = torch.zeros((n, 7), dtype=torch.int64, device="cuda")
    val = torch.zeros((n, 7), dtype=torch.float64, device="cuda")
    mask = torch.zeros((n, 7), dtype=torch.bool, device="cuda")
    col[:, 3] = idx.reshape(-1)
    val[:, 3] = diag.reshape(-1)
    mask[:, 3] = True
    stride = (shape[1] * shape[2], shape[2], 1)
    for ax, (minus, plus) in enumerate(((0, 6), (1, 5), (2, 4))):
        if faces[ax] is None or shape[ax] < 2:
            continue
        lo = idx.narrow(ax, 0, shape[ax] - 1).reshape(-1)
        t = faces[ax].narrow(ax, 0, shape[ax] - 1).reshape(-1)
        hi = lo + stride[ax]
        col[lo, plus], val[lo, plus], mask[lo, plus] = hi, -t, True
        col[hi, minus], val[hi, minus], mask[hi, minus] = lo, -t, True
    if case["problem"] == "convdiff2d":   # first-order upwind convection along x
        at = mask[:, 2]
        val[at, 2] -= 0.8
        val[at, 3] += 0.8
    return col, val, mask


def _csr(col, val, mask):
    rp = torch.zeros(col.shape[0] + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(mask.sum(dim=1), 0, out=rp[1:])
    return rp.to(torch.int32), col[mask].to(torch.int32), val[mask].contiguous()


def _product(col, val, x):
    """A x over the seven slots, in slot order (masked slots hold zeros)."""
    y = val[:, 0, None] * x[col[:, 0]] if x.dim() == 2 else val[:, 0] * x[col[:, 0]]
    for s in range(1, 7):
        y = y + (val[:, s, None] * x[col[:, s]] if x.dim() == 2 else val[:, s] * x[col[:, s]])
    return y


def _solution(n, seed, cols=0):
    g = torch.Generator(device="cuda").manual_seed(int(seed) + 7919)
    return 2.0 * torch.rand((n, cols) if cols else (n,), dtype=torch.float64, device="cuda", generator=g) - 1.0


def _batch_grids(case):
    sides = np.random.default_rng(case["layout"]).integers(case["lo"], case["hi"] + 1, size=case["nsys"])
    return [dict(problem="poisson2d", nx=int(s), ny=int(s), nz=1) for s in sides]


def _system(case, seed):
    """(slots, row offsets of the systems or None)."""
    if case["path"] != "batch":
        return _slots(case, seed), None
    off, parts = [0], []
    for grid in _batch_grids(case):
        c, v, m = _slots(grid, seed)
        parts.append((c + off[-1], v, m))
        off.append(off[-1] + c.shape[0])
    return tuple(torch.cat([p[q] for p in parts]) for q in range(3)), off


def _options(case):
    kw = {k: case[k] for k in ("krylov", "smoother", "kcycle_levels", "mis_k") if k in case}
    return amg.Options(dim=2 if case["problem"].endswith("2d") else 3, precision=case["precision"], **kw)


# ---------------------------------------------------------------- a pass


def prepare(case, seed):
    (col, val, mask), off = _system(case, seed)
    n, path = col.shape[0], case["path"]
    dev = _csr(col, val, mask)
    st = {"path": path, "dev": dev, "off": off, "opts": _options(case)}
    if path == "spmv":
        st["x"] = _solution(n, seed)
        st["y"] = torch.empty_like(st["x"])
        return st
    if path == "train":
        st["h"] = amg.setup(*dev, st["opts"])
        st["errors"] = _solution(n, seed, case["samples"])
        st["w"] = torch.from_numpy(learned.init_weights(int(seed) % 1000)).cuda()
        st["m"], st["v"], st["g"] = (torch.zeros_like(st["w"]) for _ in range(3))
        st["step"] = 0
        return st
    if path in ("solve", "multi", "resetup"):
        st["h"] = amg.setup(*dev, st["opts"])
    if path == "resetup":   # the coefficients of the next step
        col, val, mask = _slots(case, seed + 1000003)
        st["val"] = val[mask].contiguous()
    st["b"] = _product(col, val, _solution(n, seed, case.get("nrhs", 0))).contiguous()
    st["x"] = torch.empty_like(st["b"])
    return st


def run(st):
    path = st["path"]
    if path == "spmv":
        return amg.spmv(*st["dev"], st["x"], st["y"])
    if path == "train":
        st["step"] += 1
        loss = amg.mlp_loss_grad(st["h"], 0, st["w"], 0, 0, st["errors"], st["g"], raw_extra=True)
        amg.mlp_adam(st["w"], st["m"], st["v"], st["g"], st["step"], 1e-3)
        return {"loss": loss, "grad": st["g"], "w": st["w"], "m": st["m"], "v": st["v"]}
    if path == "multi":
        x, iters, _ = amg.solve_multi(st["h"], st["b"], RTOL, X=st["x"])
        return {"x": x, "iters": iters}
    if path in ("solve", "resetup"):
        if path == "resetup":
            st["h"].resetup(st["val"])
        x, iters, _ = amg.solve(st["h"], st["b"], RTOL, x=st["x"])
        return {"x": x, "iters": iters}
    h = amg.setup(*st["dev"], st["opts"]) if path == "setup_solve" else amg.setup_batched(*st["dev"], st["off"],
                                                                                            st["opts"])
    x, iters, _ = amg.solve(h, st["b"], RTOL, x=st["x"])
    out = {"x": x, "iters": h.batch_results()[0] if path == "batch" else iters}
    h.close()
    return out


# ---------------------------------------------------------------- what a pass needs


def _sizes(case):
    grids = _batch_grids(case) if case["path"] == "batch" else [case]
    n = nnz = 0
    for g in grids:
        m = g["nx"] * g["ny"] * g["nz"]
        n += m
        nnz += m + 2 * sum(m // d * (d - 1) for d in (g["nx"], g["ny"], g["nz"]))
    return n, nnz


def work(case):
    """Bytes and operations of the method.  The matrix is counted as CSR, the
    coarse levels not at all.  A set-up reads the matrix for the strength test,
    for each of five Arnoldi steps and for the coarse product; an outer
    iteration reads it for the Krylov product, the residual before the coarse
    correction and the post-smoothing, each with a vector read and one
    written."""
    n, nnz = _sizes(case)
    path, R = case["path"], case.get("nrhs", 1)
    csr = 12 * nnz + 4 * (n + 1)
    if path == "spmv":
        return {"bytes": csr + 16 * n, "flops": 2 * nnz}
    if path == "train":   # the errors, A E, A (I - W A) E, the features and one pass of the network and back
        S = case["samples"]
        return {"bytes": 2 * csr + 4 * 8 * n * S + 2 * 36 * n, "flops": n * (6 * 1376 + 40 * S)}
    it = ITERATIONS[case["problem"]]
    vb = 4 if case["precision"] == "mixed" else 8   # of the cycle's matrix and vectors
    per = csr + 16 * n * R + 2 * ((vb + 4) * nnz + 4 * (n + 1) + 2 * vb * n * R)
    setup = 0 if path in ("solve", "multi") else 7 * csr
    return {"bytes": setup + it * per, "flops": it * 6 * nnz * R + (12 * nnz if setup else 0)}


# ---------------------------------------------------------------- 64-bit results


def _bf16(x):
    return x.float().bfloat16().double()


class _Rounded(torch.autograd.Function):
    """bfloat16 rounding, passed straight through in the backward pass."""

    @staticmethod
    def forward(ctx, x):
        return _bf16(x)

    @staticmethod
    def backward(ctx, g):
        return g


def _train_exact(case, seed):
    col, val, mask = _slots(case, seed)
    n = col.shape[0]
    E = _solution(n, seed, case["samples"])
    d = val[:, 3]
    ad = d.abs()
    off = val.abs()
    off[:, 3] = 0.0
    logd = ad.log()
    ratio = torch.sort(off / ad[:, None], dim=1, descending=True).values[:, :6]
    F = torch.cat([(logd - logd.mean())[:, None], ratio, (val.sum(dim=1) / d)[:, None],
                   torch.zeros((n, 1), dtype=torch.float64, device="cuda")], dim=1)
    w0 = torch.from_numpy(learned.init_weights(int(seed) % 1000)).cuda()
    w = w0.double().requires_grad_()
    r = _Rounded.apply
    W1, b1, W2, b2, W3, b3 = torch.split(w, [288, 32, 1024, 32, 32, 1])
    h1 = r(torch.relu(_bf16(F) @ r(W1).reshape(32, 9).T + b1))
    h2 = r(torch.relu(h1 @ r(W2).reshape(32, 32).T + b2))
    y = h2 @ r(W3) + b3
    omega = torch.sigmoid(y) * 2.0 * ad / (ad + off.sum(dim=1))
    AE = _product(col, val, E)
    E2 = E - (omega / d)[:, None] * AE
    loss = ((E2 * _product(col, val, E2)).sum(dim=0) / (E * AE).sum(dim=0)).mean()
    g, = torch.autograd.grad(loss, w)
    m, v = 0.1 * g, 0.001 * g * g
    new = w0.double() - 1e-3 * g / ((v / 0.001).sqrt() + 1e-8)
    return {"loss": loss.detach(), "grad": g, "w": new, "m": m, "v": v}


def exact(case, seed):
    if case["path"] == "train":
        return _train_exact(case, seed)
    if case["path"] == "spmv":
        col, val, _ = _slots(case, seed)
        return _product(col, val, _solution(col.shape[0], seed))
    # right-hand sides are formed as A x: the solution is known
    return {"x": _solution(_sizes(case)[0], seed, case.get("nrhs", 0)), "iters": None}
