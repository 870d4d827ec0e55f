"""The library's measured workloads: ghost exchange, redistribution and every solver form, over its range of sizes.

A case is a dict of plain values; `prepare` makes its inputs and handles on
the GPU, `run` makes one pass through the public entry points, `work` gives
the bytes and operations a pass cannot do without, and `exact` the result in
64 bits from plain torch (1-D eigendecompositions for constant coefficients,
conjugate gradients preconditioned with them for variable ones).

Kinds
  fill       FillBoundary (and the physical ghosts of a domain with Dirichlet
             faces) on a MultiFab: what an explicit stencil code calls once
             per stage, so its latency counts at small sizes
  copy       ParallelCopy onto another decomposition, ghosts included
  solve      one cell-centred solve from a zero guess
  heat       one backward-Euler heat step with a source
  nodal      one nodal solve from a zero guess
  composite  one two-level solve (central half refined by 2)
  batch      many periodic or many variable-coefficient problems solved
             together by the batch engine
"""
import math

import numpy as np
import torch

import paper_2403_12179_amd as bx

TOL = 1e-10  # the tolerance the library's benchmark solves to


def listed():
    return [
        # an explicit code's exchange on a small periodic patch: launch latency
        dict(name="fill_48_periodic", kind="fill", nx=48, ny=48, nz=48, box=32, nghost=1, ncomp=1, dtype="f64",
             periodic="111"),
        # a large single-precision state of two components with two ghost
        # layers in the 512-box decomposition, Dirichlet domain
        dict(name="fill_256_f32_dirichlet", kind="fill", nx=256, ny=256, nz=256, box=32, nghost=2, ncomp=2,
             dtype="f32", periodic="000"),
        # redistribution of a ragged domain between two decompositions
        dict(name="copy_208_regrid", kind="copy", nx=208, ny=176, nz=240, box=64, box_to=32, nghost=1, ncomp=1,
             dtype="f64", periodic="101"),
        # the smallest solve in use: one box, latency-bound
        dict(name="solve_32_periodic", kind="solve", nx=32, ny=32, nz=32, box=32, periodic="111", precision=0,
             krylov=0, var=False, rel_tol=TOL),
        # a ragged mid-size domain, mixed boundaries, odd bottom level
        dict(name="solve_96x48x80_mixed", kind="solve", nx=96, ny=48, nz=80, box=32, periodic="101", precision=0,
             krylov=0, var=False, rel_tol=TOL),
        # a served request with a variable coefficient, mixed precision
        dict(name="solve_128_varcoef_mixed", kind="solve", nx=128, ny=128, nz=128, box=32, periodic="000",
             precision=1, krylov=0, var=True, rel_tol=1e-9),
        # the benchmark's headline problem
        dict(name="solve_256_dirichlet", kind="solve", nx=256, ny=256, nz=256, box=32, periodic="000", precision=0,
             krylov=0, var=False, rel_tol=TOL),
        # the largest: variable coefficient, CG preconditioned by a V-cycle
        # in single precision
        dict(name="solve_512_varcoef_pcg", kind="solve", nx=512, ny=512, nz=512, box=64, periodic="000", precision=1,
             krylov=1, var=True, rel_tol=TOL),
        # a time step of the heat equation with a source
        dict(name="heat_192_source", kind="heat", nx=192, ny=192, nz=192, box=32, periodic="000", dt=1e-4,
             rel_tol=TOL),
        # the benchmark's nodal problem
        dict(name="nodal_256_dirichlet", kind="nodal", nx=256, ny=256, nz=256, periodic="000", rel_tol=TOL),
        # the benchmark's two-level problem
        dict(name="composite_256", kind="composite", n=256, box=32, periodic="000", rel_tol=TOL),
        # a batch of independent periodic problems, mixed precision
        dict(name="batch_64_periodic_mixed", kind="batch", count=64, edges_seed=4, periodic="111", precision=1,
             var=False, rel_tol=TOL),
    ]


def draw(rng):
    """A case of one kind with sizes, boundaries and options over the ranges."""
    def edge(lo, hi, step):  # a multiple of step, spread over the logarithm
        return max(lo, min(hi, step * round(math.exp(rng.uniform(math.log(lo), math.log(hi))) / step)))

    def per():
        return rng.choice(["000", "111", "101", "010", "110"])

    kind = rng.choice(["fill", "copy", "solve", "solve", "solve", "heat", "nodal", "composite", "batch"])
    if kind in ("fill", "copy"):
        box, to = rng.choice([16, 32, 64]), rng.choice([16, 24, 32, 48, 64])
        while True:  # ragged edges, odd ones too, whose boxes stay wider than the ghost layers
            n = [edge(12, 272, 1) for _ in range(3)]
            if all(min(_pieces(e, b)) >= 4 for e in n for b in (box, to)):
                break
        c = dict(kind=kind, nx=n[0], ny=n[1], nz=n[2], box=box, nghost=rng.randint(1, 3), ncomp=rng.randint(1, 2),
                 dtype=rng.choice(["f64", "f32"]), periodic=per())
        if kind == "copy":
            c["box_to"] = to
        return c
    if kind == "solve":
        n = [edge(32, 256, 16) for _ in range(3)]
        if rng.random() < 0.5:
            n = [n[0]] * 3
        return dict(kind="solve", nx=n[0], ny=n[1], nz=n[2], box=rng.choice([32, 64]), periodic=per(),
                    precision=rng.randint(0, 1), krylov=rng.randint(0, 1), var=rng.random() < 0.4,
                    rel_tol=10.0 ** rng.uniform(-10.0, -8.0))
    if kind == "heat":
        n = edge(32, 256, 16)
        return dict(kind="heat", nx=n, ny=n, nz=n, box=32, periodic=per(), dt=10.0 ** rng.uniform(-5.0, -3.0),
                    rel_tol=TOL)
    if kind == "nodal":
        n = [edge(32, 256, 16) for _ in range(3)]
        return dict(kind="nodal", nx=n[0], ny=n[1], nz=n[2], periodic=per(), rel_tol=TOL)
    if kind == "composite":
        return dict(kind="composite", n=edge(32, 256, 32), box=rng.choice([16, 32]), periodic="000", rel_tol=TOL)
    var = rng.random() < 0.3
    return dict(kind="batch", count=rng.randint(4, 16 if var else 64), edges_seed=rng.randint(0, 10 ** 6),
                periodic="000" if var else "111", precision=rng.randint(0, 1), var=var,
                rel_tol=10.0 ** rng.uniform(-10.0, -8.0))


# ------------------------------------------------------------- geometry
def _shape(case):
    return (case["nx"], case["ny"], case["nz"]) if "nx" in case else (case["n"],) * 3


def _bc(periodic):
    return tuple(bx.PERIODIC if c == "1" else bx.DIRICHLET0 for c in periodic)


def _pieces(n, box):
    """Edge lengths a domain edge n is chopped into (include/bxmg.h)."""
    bf = 1
    while n % (2 * bf) == 0 and 2 * bf <= box:
        bf *= 2
    p = box // bf * bf
    return [p] * (n // p) + ([n % p] if n % p else [])


def _boxes(shape, box):
    """(lo, size) of the boxes of a chopped domain, x fastest."""
    cuts = []
    for n in shape:
        at, c = 0, []
        for p in _pieces(n, box):
            c.append((at, p))
            at += p
        cuts.append(c)
    return [((i[0], j[0], k[0]), (i[1], j[1], k[1])) for k in cuts[2] for j in cuts[1] for i in cuts[0]]


def _slab(boxes, nghost, comps, esize, ghosts):
    """The flat slab of a MultiFab whose box b holds comps[c](lo, hi) on its
    grown (ghosts) or valid cells and 0 elsewhere; boxes start at 256 B."""
    parts = []
    for lo, size in boxes:
        g = nghost if ghosts else 0
        for field in comps:
            v = field(tuple(a - g for a in lo), tuple(a + s + g for a, s in zip(lo, size)))
            if not ghosts:
                v = np.pad(v, nghost)
            parts.append(v.ravel(order="F"))
        n = len(comps) * math.prod(s + 2 * nghost for s in size)
        parts.append(np.zeros(-n % (256 // esize), parts[-1].dtype))
    return np.concatenate(parts)


def _ba(shape, box, periodic):
    return bx.BoxArray.chop((0, 0, 0), tuple(n - 1 for n in shape), box, bc=_bc(periodic))


# --------------------------------------------------------------- inputs
def _uniform(shape, seed, mean_zero=False, dtype=torch.float64):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) & 0x7FFFFFFFFFFFFFFF)
    f = torch.rand(tuple(shape), generator=g, device="cuda", dtype=torch.float64) * 2.0 - 1.0
    return (f - f.mean() if mean_zero else f).to(dtype)


def _beta(shape, seed):
    """exp of smoothed Gaussian noise of mean 0 and deviation 1."""
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) & 0x7FFFFFFFFFFFFFFF)
    x = torch.randn(tuple(shape), generator=g, device="cuda", dtype=torch.float64)
    for _ in range(3):
        for d in range(3):
            x = (x + torch.roll(x, 1, d) + torch.roll(x, -1, d)) / 3.0
    return torch.exp((x - x.mean()) / x.std(unbiased=False))


def _mf(ba, field, nghost=1):
    return bx.MultiFab(ba, nghost=nghost).set_val(0.0).from_tensor(field)


def _seed(case, seed, part):
    return (int(seed) * 1000003 + part * 7919) % (1 << 62)


def _rhs(case, seed):
    """Right-hand side; compatible (mean zero) where the operator is singular."""
    return _uniform(_shape(case), _seed(case, seed, 1), case["periodic"] == "111" and case["kind"] == "solve")


def _nodal_rhs(case, seed):
    """[k, j, i] node values; periodic directions repeat node 0 at node n."""
    n = _shape(case)
    f = _uniform((n[2] + 1, n[1] + 1, n[0] + 1), _seed(case, seed, 1))
    if case["periodic"] == "111":
        f -= f[:-1, :-1, :-1].mean()
    for d in range(3):
        if case["periodic"][d] == "1":
            f.select(2 - d, n[d]).copy_(f.select(2 - d, 0))
    return f


def _batch_edges(case):
    return np.random.default_rng(case["edges_seed"]).choice((32, 48, 64, 96, 128), size=case["count"])


def _batch_fields(case, seed, p, e):
    f = _uniform((e,) * 3, _seed(case, seed, 10 + p), case["periodic"] == "111")
    return f, _beta((e,) * 3, _seed(case, seed, 5000 + p)) if case["var"] else None


def _composite_boxes(case):
    n, b = case["n"], case["box"]
    lo, hi = 2 * (n // 4), 2 * (n - n // 4)
    at = range(lo, hi, b)
    return [((i, j, k), tuple(min(a + b, hi) - 1 for a in (i, j, k))) for k in at for j in at for i in at]


# ------------------------------------------------------------------ api
def prepare(case, seed):
    kind, shape = case["kind"], _shape(case) if case["kind"] != "batch" else None
    if kind in ("fill", "copy"):
        dt = torch.float64 if case["dtype"] == "f64" else torch.float32
        src = bx.MultiFab(_ba(shape, case["box"], case["periodic"]), ncomp=case["ncomp"],
                          nghost=case["nghost"] if kind == "fill" else 0, dtype=case["dtype"]).set_val(0.0)
        for c in range(case["ncomp"]):
            src.from_tensor(_uniform(shape, _seed(case, seed, 1 + c), dtype=dt), comp=c)
        if kind == "fill":
            return dict(case=case, mf=src)
        dst = bx.MultiFab(_ba(shape, case["box_to"], case["periodic"]), ncomp=case["ncomp"], nghost=case["nghost"],
                          dtype=case["dtype"]).set_val(0.0)
        return dict(case=case, src=src, mf=dst)
    if kind == "solve":
        ba = _ba(shape, case["box"], case["periodic"])
        return dict(case=case, phi=_mf(ba, torch.zeros(1, device="cuda").double().expand(shape)),
                    rhs=_mf(ba, _rhs(case, seed)),
                    beta=_mf(ba, _beta(shape, _seed(case, seed, 2))) if case["var"] else None,
                    par=dict(precision=case["precision"], krylov=case["krylov"], rel_tol=case["rel_tol"]))
    if kind == "heat":
        ba = _ba(shape, case["box"], case["periodic"])
        u0 = _mf(ba, _uniform(shape, _seed(case, seed, 3)))
        return dict(case=case, u0=u0, u=bx.MultiFab(ba).set_val(0.0), source=_mf(ba, _rhs(case, seed)))
    if kind == "nodal":
        rhs = _nodal_rhs(case, seed)
        return dict(case=case, ba=_ba(shape, 32, case["periodic"]), rhs=rhs, phi=torch.zeros_like(rhs))
    if kind == "composite":
        n = case["n"]
        cba = _ba(shape, 32, case["periodic"])
        fba = bx.BoxArray.from_boxes((0, 0, 0), (2 * n - 1,) * 3, _composite_boxes(case), bc=_bc(case["periodic"]))
        return dict(case=case, pc=bx.MultiFab(cba).set_val(0.0), pf=bx.MultiFab(fba).set_val(0.0),
                    rc=_mf(cba, _uniform(shape, _seed(case, seed, 1)), nghost=0),
                    rf=_mf(fba, _uniform((2 * n,) * 3, _seed(case, seed, 2)), nghost=0))
    probs = []
    for p, e in enumerate(_batch_edges(case)):
        e = int(e)
        ba = _ba((e,) * 3, 32, case["periodic"])
        f, beta = _batch_fields(case, seed, p, e)
        probs.append((bx.MultiFab(ba).set_val(0.0), _mf(ba, f), _mf(ba, beta) if case["var"] else None))
    ctx = bx.default_context()
    batch = bx.Batch(ctx, 6 << 30, case["count"], var=case["var"], precision=case["precision"])
    return dict(case=case, probs=probs, batch=batch)


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "fill":
        mf = state["mf"].fill_boundary()
        if "0" in case["periodic"]:
            mf.apply_domain_bc()
        return mf.slab
    if kind == "copy":
        return state["mf"].parallel_copy(state["src"], nghost=case["nghost"]).slab
    if kind == "solve":
        phi = state["phi"].set_val(0.0)
        bx.mlmg_solve(phi, state["rhs"], state["beta"], **state["par"])
        return phi.slab
    if kind == "heat":
        u = state["u"]
        u.slab.copy_(state["u0"].slab)
        bx.heat_step(u, case["dt"], source=state["source"], rel_tol=case["rel_tol"])
        return u.slab
    if kind == "nodal":
        phi = state["phi"].zero_()
        bx.nodal_solve(state["ba"], phi, state["rhs"], rel_tol=case["rel_tol"])
        return phi
    if kind == "composite":
        bx.composite_solve(state["pc"], state["rc"], state["pf"], state["rf"], rel_tol=case["rel_tol"])
        return [state["pc"].slab, state["pf"].slab]
    batch = state["batch"]
    for phi, rhs, beta in state["probs"]:
        if batch.add(phi.set_val(0.0), rhs, beta, rel_tol=case["rel_tol"]) is None:
            raise RuntimeError("the batch's arena is too small for its problems")
    batch.run(2)
    return [phi.slab for phi, _, _ in state["probs"]]


#: Operations per fine cell and V(2,2) cycle: four sweeps of 8, the two
#: residuals of 9 and the correction's 8, times 8/7 for the coarser levels.
CYCLE_FLOPS = 66
#: Cycles from a zero guess to 1e-10, as the iteration contracts: constant
#: coefficient, variable coefficient, the latter with CG.
CYCLES = {False: 10, True: 35, "krylov": 17}


def work(case):
    """Inputs once, outputs once; the operations of the cycles the iteration
    takes.  fill: the ghost cells' values read and written; copy: each
    destination cell read and written."""
    kind = case["kind"]
    if kind in ("fill", "copy"):
        es, g = (8 if case["dtype"] == "f64" else 4) * case["ncomp"], case["nghost"]
        cells = 0
        for _, s in _boxes(_shape(case), case["box" if kind == "fill" else "box_to"]):
            cells += math.prod(a + 2 * g for a in s) - (math.prod(s) if kind == "fill" else 0)
        return {"bytes": 2 * es * cells, "flops": 0}
    if kind == "batch":
        cells = sum(int(e) ** 3 for e in _batch_edges(case))
        return {"bytes": 8 * cells * (4 if case["var"] else 3), "flops": cells * CYCLE_FLOPS * CYCLES[case["var"]]}
    cells = math.prod(_shape(case))
    if kind == "composite":  # both levels start from zero
        return {"bytes": 2 * 8 * 2 * cells, "flops": 2 * cells * CYCLE_FLOPS * CYCLES[False]}
    if kind == "solve":
        cycles = CYCLES["krylov"] if case["krylov"] and case["var"] else CYCLES[case["var"]]
        return {"bytes": 8 * cells * (4 if case["var"] else 3), "flops": cells * CYCLE_FLOPS * cycles}
    return {"bytes": 3 * 8 * cells, "flops": cells * CYCLE_FLOPS * (7 if kind == "heat" else CYCLES[False])}


# ---------------------------------------------------------------- exact
def _extended(t, periodic, g, odd):
    """t grown by g: periodic images, odd reflection (or zeros) elsewhere."""
    for d in range(3):
        n = t.shape[d]
        at = np.arange(-g, n + g)
        if periodic[d] == "1":
            t = np.take(t, at % n, axis=d)
        else:
            out = (at < 0) | (at >= n)
            m = np.where(at < 0, -1 - at, np.where(at >= n, 2 * n - 1 - at, at))
            s = np.where(out, -1.0 if odd else 0.0, 1.0).astype(t.dtype)
            t = np.take(t, m, axis=d) * s.reshape([-1 if k == d else 1 for k in range(3)])
    return t


def _eig(n, periodic, nodal=False):
    """Eigenvalues and vectors of the 1-D second difference (h = 1)."""
    m = n - 1 if nodal and not periodic else n
    a = torch.diag(torch.full((m,), -2.0, dtype=torch.float64))
    i = torch.arange(m - 1)
    a[i, i + 1] = 1.0
    a[i + 1, i] = 1.0
    if periodic:
        a[0, m - 1] += 1.0
        a[m - 1, 0] += 1.0
    elif not nodal:
        a[0, 0] -= 1.0
        a[m - 1, m - 1] -= 1.0
    w, v = torch.linalg.eigh(a)
    return w, v


class _Direct:
    """(L - alpha)^-1 of the constant-coefficient operator of cell width h."""

    def __init__(self, shape, periodic, h, alpha=0.0, nodal=False, device="cpu"):
        eig = [_eig(n, p == "1", nodal) for n, p in zip(shape, periodic)]
        self.v = [v.to(device) for _, v in eig]
        w = [x.to(device) for x, _ in eig]
        lam = (w[0][:, None, None] + w[1][None, :, None] + w[2][None, None, :]) / (h * h) - alpha
        small = lam.abs() < 1e-9 / (h * h) if alpha == 0.0 else torch.zeros_like(lam, dtype=torch.bool)
        self.inv = torch.where(small, torch.zeros_like(lam), 1.0 / torch.where(small, torch.ones_like(lam), lam))

    def _apply(self, t, back):
        for d in range(3):
            m = self.v[d] if back else self.v[d].t().contiguous()
            t = torch.movedim(torch.mm(m, torch.movedim(t, d, 0).reshape(m.shape[1], -1))
                              .reshape([m.shape[0]] + [t.shape[k] for k in range(3) if k != d]), 0, d)
        return t

    def __call__(self, f):
        return self._apply(self._apply(f, False) * self.inv, True)


def _var_solve(f, beta, periodic, h):
    """Conjugate gradients on div(beta grad u) = f with harmonic faces,
    preconditioned by beta^-1/2 (laplacian)^-1 beta^-1/2."""
    def shift(t, d, by, ghost):  # t at the neighbour, `ghost` times the cell itself beyond a Dirichlet face
        s = torch.roll(t, -by, d)
        if periodic[d] != "1":
            k = t.shape[d] - 1 if by > 0 else 0
            s.select(d, k).copy_(t.select(d, k) * ghost)
        return s

    faces = [(d, by, 2.0 * beta * b / (beta + b)) for d in range(3) for by in (-1, 1)
             for b in [shift(beta, d, by, 1.0)]]
    sb = sum(b for _, _, b in faces)

    def op(u):  # minus the operator: positive definite
        q = sb * u
        for d, by, b in faces:
            q -= b * shift(u, d, by, -1.0)
        return q / (h * h)

    singular = periodic == "111"
    direct, rb = _Direct(f.shape, periodic, h, device=f.device), beta.rsqrt()
    u, r = torch.zeros_like(f), -f
    p, rz = None, None
    stop = 1e-13 * float(f.norm())
    for _ in range(3000):
        z = -rb * direct(rb * r)
        new = float((r * z).sum())
        p = z if p is None else z + (new / rz) * p
        rz = new
        q = op(p)
        a = rz / float((p * q).sum())
        u += a * p
        r -= a * q
        if float(r.norm()) <= stop:
            break
    return u - u.mean() if singular else u


def _solved(case, shape, f, beta):
    h = 1.0 / shape[0]
    u = _var_solve(f, beta, case["periodic"], h) if beta is not None else \
        _Direct(shape, case["periodic"], h, device=f.device)(f)
    return u.cpu().numpy()


def _valid(t):
    return lambda lo, hi: t[tuple(slice(a, b) for a, b in zip(lo, hi))]


def exact(case, seed):
    kind = case["kind"]
    if kind == "composite":  # two coupled levels: no fast direct solve
        return None
    if case.get("var") and kind == "solve" and math.prod(_shape(case)) > 1 << 22:
        return None  # thousands of iterations: longer than 20 s
    if kind in ("fill", "copy"):
        shape, g, es = _shape(case), case["nghost"], 8 if case["dtype"] == "f64" else 4
        dt = torch.float64 if es == 8 else torch.float32
        grown = []
        for c in range(case["ncomp"]):
            t = _extended(_uniform(shape, _seed(case, seed, 1 + c), dtype=dt).cpu().numpy(), case["periodic"], g,
                          kind == "fill")
            grown.append(lambda lo, hi, t=t: t[tuple(slice(a + g, b + g) for a, b in zip(lo, hi))])
        return _slab(_boxes(shape, case["box" if kind == "fill" else "box_to"]), g, grown, es, True)
    if kind == "solve":
        shape = _shape(case)
        u = _solved(case, shape, _rhs(case, seed), _beta(shape, _seed(case, seed, 2)) if case["var"] else None)
        return _slab(_boxes(shape, case["box"]), 1, [_valid(u)], 8, False)
    if kind == "heat":
        shape = _shape(case)
        f = -(_uniform(shape, _seed(case, seed, 3)) / case["dt"] + _rhs(case, seed))
        u = _Direct(shape, case["periodic"], 1.0 / shape[0], 1.0 / case["dt"], device=f.device)(f).cpu().numpy()
        return _slab(_boxes(shape, case["box"]), 1, [_valid(u)], 8, False)
    if kind == "nodal":
        n = _shape(case)
        f = _nodal_rhs(case, seed)
        inner = tuple(slice(0, m) if p == "1" else slice(1, m)
                      for m, p in zip((n[2], n[1], n[0]), case["periodic"][::-1]))
        u = torch.zeros_like(f)
        u[inner] = _Direct(n[::-1], case["periodic"][::-1], 1.0 / n[0], nodal=True, device=f.device)(f[inner])
        for d in range(3):
            if case["periodic"][d] == "1":
                u.select(2 - d, n[d]).copy_(u.select(2 - d, 0))
        return u.cpu().numpy()
    out = []
    for p, e in enumerate(_batch_edges(case)):
        e = int(e)
        f, beta = _batch_fields(case, seed, p, e)
        out.append(_slab(_boxes((e,) * 3, 32), 1, [_valid(_solved(case, (e,) * 3, f, beta))], 8, False))
    return out
