"""Timed cases of the library: the calls a Stokes solve is made of, each
through the public entry points of paper_2010_13513_amd.hhg.

Every case is a dict of plain values; `prepare` builds what a program holds
before the call (hierarchy, vectors), `run` makes one pass, `exact` evaluates
the same in float64 with plain torch / numpy from the finite-element
definitions.  Sizes are the repository's own: 6 or 48 Kuhn macro-tetrahedra
(macro 0 / 1, N = 2^(level + macro) intervals per edge), the 24-tetrahedron
cube and boxes of such cubes, and the network of the learned coarse solve.
"""
import itertools
import math

import numpy as np
import torch

from paper_2010_13513_amd import hhg, workloads

DEV = "cuda:0"
F64, F32 = hhg.HHG_F64, hhg.HHG_F32
OPS = {"full": hhg.HHG_OP_FULL, "A": hhg.HHG_OP_A, "BT": hhg.HHG_OP_BT, "B": hhg.HHG_OP_B, "C": hhg.HHG_OP_C,
       "mass": hhg.HHG_OP_MASS}


# ------------------------------------------------------------------ cases
def listed():
    smooth = dict(kind="smooth", prec="f64", schur="sd", gs="f")
    return [
        # the smallest whole solve: FMG to level 3 (2916 unknowns), latency only
        dict(name="fmg_p1_l3", kind="fmg", disc=1, macro=0, lmin=0, level=3, pre=2, post=3, inc=2, kappa=1, gs="s",
             xi=1, omega_inv=2.30),
        # the benchmark's solve: Taylor-Hood FMG(1,3,0,1,A_f,3) to level 5 (859,812 unknowns)
        dict(name="fmg_p2_l5", kind="fmg", disc=2, macro=0, lmin=1, level=5, pre=1, post=3, inc=0, kappa=1, gs="f",
             xi=3, omega_inv=2.34),
        # the smoothing inside that solve on a middle level: three Uzawa iterations
        dict(name="smooth_p2_l4", disc=2, macro=0, level=4, iters=3, xi=3, **smooth),
        # P1-P1 smoothing on the level of its own benchmark solve (1,098,500 unknowns)
        dict(name="smooth_p1_l6", disc=1, macro=0, level=6, iters=1, xi=3, **smooth),
        # an Uzawa iteration of the throughput sweep at its largest size (3.5e8 unknowns)
        dict(name="smooth_p2_48_l7", disc=2, macro=1, level=7, iters=1, xi=3, **smooth),
        # the same in float32 one level below, symmetric sweep: the inner cycles of defect correction
        dict(name="smooth_p2_48_l6_f32", disc=2, macro=1, level=6, iters=1, xi=1, **{**smooth, "prec": "f32", "gs": "s"}),
        # the operator apply of the roofline measurement
        dict(name="apply_p2_48_l7", kind="apply", op="full", disc=2, macro=1, level=7, prec="f64"),
        # the residual of a P1-P1 cycle in float32, largest level of the sweep
        dict(name="residual_p1_48_l7_f32", kind="apply", op="residual", disc=1, macro=1, level=7, prec="f32"),
        # both grid transfers of a cycle, down and up
        dict(name="transfer_p2_48_l6", kind="transfer", disc=2, macro=1, level=6, prec="f64"),
        # one V(3,3) in float32 with variable viscosity: the inner cycle of mixed-precision defect correction
        dict(name="vcycle_p2_visc_l6_f32", kind="vcycle", disc=2, macro=0, lmin=1, level=6, prec="f32", visc=True, pre=3,
             post=3, inc=0, gs="f", xi=3, omega_inv=2.4),
        # the paper's cube benchmark on an unstructured mesh: FMG on 24 tetrahedra, level 6 (4,293,636 unknowns)
        dict(name="umesh_fmg_l6", kind="umesh_fmg", boxes=1, level=6, pre=2, post=3, inc=2, kappa=1, gs="s", xi=1,
             omega_inv=2.69),
        # training the learned coarse solve: an epoch of minibatches, 331 -> 512 -> 512 -> 512 -> 206
        dict(name="mlp_train", kind="mlp_train", n_in=331, hidden=512, n_out=206, samples=20000, batch=256, epochs=1),
    ]


def draw(rng):
    """A case of the listed ones' ranges: any discretisation, precision, level,
    option and mesh that costs no more than the largest listed one."""
    kind = rng.choice(["fmg", "smooth", "smooth", "apply", "transfer", "vcycle", "umesh_fmg", "umesh_smooth",
                       "mlp_train"])
    disc = rng.choice([1, 2])
    macro = rng.choice([0, 1])
    prec = rng.choice(["f64", "f32"])
    gs = rng.choice(["f", "s"])
    if kind == "fmg":
        lmin = rng.choice([0, 1]) if disc == 1 else 1 - macro
        return dict(kind=kind, disc=disc, macro=macro, lmin=lmin, level=rng.randint(2, (6 if disc == 1 else 5) - macro),
                    pre=rng.randint(0, 2), post=rng.randint(1, 3), inc=rng.randint(0, 2), kappa=rng.choice([1, 1, 2]),
                    gs=gs, xi=rng.randint(1, 3) if gs == "f" else 1, omega_inv=2.3)
    if kind == "smooth":
        level = rng.randint(2, 7)
        big = disc == 2 and level + macro >= 7
        sweeps = rng.randint(1, 3)
        gs = "f" if big else gs
        return dict(kind=kind, disc=disc, macro=macro, level=level, prec=prec, schur=rng.choice(["sd", "ml"]), gs=gs,
                    iters=1 if level + macro >= 7 else rng.randint(1, 3), xi=sweeps if gs == "f" else rng.randint(1, 2))
    if kind == "apply":
        op = rng.choice(["full", "residual", "residual", "A", "BT", "B", "mass"] + (["C"] if disc == 1 else []))
        return dict(kind=kind, op=op, disc=disc, macro=macro, level=rng.randint(2, 7), prec=prec)
    if kind == "transfer":
        return dict(kind=kind, disc=disc, macro=macro, level=rng.randint(3, 7), prec=prec)
    if kind == "vcycle":
        visc = rng.random() < 0.5
        return dict(kind=kind, disc=disc, macro=0, lmin=1, level=rng.randint(2, 6), prec=prec, visc=visc,
                    pre=rng.randint(0, 3), post=rng.randint(1, 3), inc=rng.randint(0, 1), gs="f",
                    xi=rng.randint(1, 3) if disc == 1 else 3, omega_inv=2.4)
    if kind == "mlp_train":
        return dict(kind=kind, n_in=331, hidden=16 * rng.randint(8, 32), n_out=206,
                    samples=int(1000 * 20 ** rng.random()), batch=rng.randint(64, 256), epochs=1)
    boxes = rng.randint(1, 4)
    if kind == "umesh_smooth":
        return dict(kind=kind, boxes=boxes, level=rng.randint(2, 6 if boxes == 1 else 5), gs=gs, xi=rng.randint(1, 2),
                    iters=rng.randint(1, 3))
    return dict(kind=kind, boxes=boxes, level=rng.randint(2, 6 if boxes == 1 else 4), pre=rng.randint(0, 2),
                post=rng.randint(1, 3), inc=rng.randint(0, 2), kappa=1, gs=gs, xi=1, omega_inv=2.69)


# ----------------------------------------------------------------- inputs
def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed))


def _normal(shape, seed):
    return torch.randn(shape, generator=_gen(seed), dtype=torch.float64, device=DEV)


def _field(seed, xyz, comps, modes=6):
    """A smooth seeded field, `comps` sums of sines at the points xyz (3 tensors)."""
    r = np.random.default_rng([13513, int(seed)])
    out = [torch.zeros_like(xyz[0]) for _ in range(comps)]
    for _ in range(modes):
        k = r.integers(-3, 4, 3).astype(float)
        amp, ph = r.standard_normal(comps) / (1.0 + float(k @ k)), r.uniform(0, 2 * math.pi)
        s = torch.sin(2 * math.pi * (k[0] * xyz[0] + k[1] * xyz[1] + k[2] * xyz[2]) + ph)
        for c in range(comps):
            out[c] += float(amp[c]) * s
    return torch.stack(out)


def _grid(M):
    t = torch.arange(M + 1, dtype=torch.float64, device=DEV) / M
    z, y, x = torch.meshgrid(t, t, t, indexing="ij")
    return x, y, z


def _nodal(disc, N, seed, comps=3):
    """Nodal values of a seeded field on the velocity lattice (lattice order)."""
    return _field(seed, _grid(N if disc == 1 else 2 * N), comps)


def _nu(seed, N):
    """Nodal viscosity, contrast about 1:100."""
    g = _field(seed + 77, _grid(N), 1, modes=8)[0]
    t = _field(seed + 77, _grid(16), 1, modes=8)[0]
    return torch.exp(math.log(100.0) * (g - t.min()) / (t.max() - t.min()))


def _random_lattice(disc, N, seed):
    m = (N if disc == 1 else 2 * N) + 1
    return _normal(3 * m ** 3 + (N + 1) ** 3, seed)


def _u_values(n, seed, level, k, comps):
    """Seeded normal values of the first `comps` fields of an unstructured level, zeros after."""
    return torch.cat([_normal(comps * n, 1000 * seed + 10 * level + k),
                      torch.zeros((4 - comps) * n, dtype=torch.float64, device=DEV)])


def _boxes_mesh(boxes):
    nx, ny, nz = {1: (1, 1, 1), 2: (2, 1, 1), 3: (3, 1, 1), 4: (2, 2, 1)}[boxes]
    return workloads.cube24() if boxes == 1 else workloads.box_cube24(nx, ny, nz)


class Problem:
    """A context and a hierarchy on it, given back with the object."""

    def __init__(self, case, lmin, lmax):
        self.ctx = hhg.hhg_ctx_create(0, torch.cuda.current_stream().cuda_stream)
        if case["kind"].startswith("umesh"):
            mesh, disc = hhg.hhg_mesh_create(self.ctx, *_boxes_mesh(case["boxes"])), hhg.HHG_P1P1
        else:
            mesh = hhg.hhg_mesh_cube(self.ctx, case["macro"])
            disc = hhg.HHG_P1P1 if case["disc"] == 1 else hhg.HHG_P2P1
        schur = hhg.HHG_SCHUR_ML if case.get("schur") == "ml" else hhg.HHG_SCHUR_SD
        self.h = hhg.hhg_hier_create(mesh, disc, lmin, lmax, schur)
        hhg.hhg_mesh_destroy(mesh)
        self.lmin, self.lmax = lmin, lmax
        self.prec = F32 if case.get("prec") == "f32" else F64
        self.dtype = torch.float32 if self.prec == F32 else torch.float64

    def zeros(self, level):
        return torch.zeros(hhg.hhg_vec_layout(self.h, level)[2], dtype=self.dtype, device=DEV)

    def vec(self, level, lattice):
        v = self.zeros(level)
        hhg.hhg_vec_from_lattice(self.h, level, lattice, v, self.prec)
        return v

    def close(self):
        if self.h is not None:
            hhg.hhg_hier_destroy(self.h)
            hhg.hhg_ctx_destroy(self.ctx)
            self.h = None

    def __del__(self):
        try:
            self.close()
        except Exception:
            pass


class Trainer:
    """A network and its context, given back with the object."""

    def __init__(self, case, params):
        self.ctx = hhg.hhg_ctx_create(0, torch.cuda.current_stream().cuda_stream)
        self.m = hhg.hhg_mlp_create(self.ctx, case["n_in"], case["hidden"], case["n_out"], max(256, case["batch"]))
        hhg.hhg_mlp_set_params(self.m, params)

    def close(self):
        if self.m is not None:
            hhg.hhg_mlp_destroy(self.m)
            hhg.hhg_ctx_destroy(self.ctx)
            self.m = None

    def __del__(self):
        try:
            self.close()
        except Exception:
            pass


def _mlp_data(case, seed):
    r = np.random.default_rng([13513, int(seed)])
    dims = [case["n_in"], case["hidden"], case["hidden"], case["hidden"], case["n_out"]]
    params = []
    for i, o in zip(dims, dims[1:]):
        params += [r.uniform(-1, 1, (o, i)) * math.sqrt(6.0 / i), np.zeros(o)]
    x = _normal((case["samples"], case["n_in"]), seed).float()
    w = _normal((case["n_in"], case["n_out"]), seed + 1) / math.sqrt(case["n_in"])
    y = (x.double() @ w).float()
    order = np.concatenate([r.permutation(case["samples"]) for _ in range(case["epochs"])]).astype(np.int32)
    return params, x, y, order


def _params(case):
    gs = hhg.HHG_GS_SYM if case["gs"] == "s" else hhg.HHG_GS_FWD
    return hhg.solver_params(case["pre"], case["post"], case["inc"], case.get("kappa", 1), gs, case["xi"],
                             case["omega_inv"])


# -------------------------------------------------------- prepare and run
def prepare(case, seed):
    kind = case["kind"]
    if kind == "mlp_train":
        params, x, y, order = _mlp_data(case, seed)
        t = Trainer(case, np.concatenate([p.ravel() for p in params]).astype(np.float32))
        return dict(case=case, t=t, x=x, y=y, order=order)
    level = case["level"]
    umesh = kind.startswith("umesh")
    if kind in ("fmg", "vcycle", "umesh_fmg"):
        P = Problem(case, case.get("lmin", 0), level)
    else:
        P = Problem(case, level - 1, level)
    s = dict(case=case, P=P, prm=_params(case) if "pre" in case else None)
    if umesh:
        n = {l: hhg.hhg_vec_layout(P.h, l)[3] // 4 for l in range(P.lmin, P.lmax + 1)}

        def values(l, k, comps):
            return _u_values(n[l], seed, l, k, comps)
        s["out"] = torch.empty(4 * n[level], dtype=torch.float64, device=DEV)
        if kind == "umesh_smooth":
            s["x"], s["b"] = P.vec(level, values(level, 0, 4)), P.vec(level, values(level, 1, 4))
        else:
            s["x"] = P.vec(level, values(level, 0, 3) * 0.1)
            s["bs"] = []
            for l in range(P.lmin, P.lmax + 1):
                f, b = P.vec(l, values(l, 1, 3)), P.zeros(l)
                hhg.hhg_rhs(P.h, l, f, b)
                s["bs"].append(b)
        return s
    disc, N = case["disc"], 2 ** (level + case["macro"])
    if kind == "fmg":
        p0 = torch.zeros((N + 1) ** 3, dtype=torch.float64, device=DEV)
        s["x"] = P.vec(level, torch.cat([_nodal(disc, N, seed).reshape(-1), p0]))
        s["bs"] = []
        for l in range(P.lmin, P.lmax + 1):
            n = 2 ** (l + case["macro"])
            f = P.vec(l, torch.cat([_nodal(disc, n, seed + 1).reshape(-1) * 50.0,
                                    torch.zeros((n + 1) ** 3, dtype=torch.float64, device=DEV)]))
            b = P.zeros(l)
            hhg.hhg_rhs(P.h, l, f, b)
            s["bs"].append(b)
        return s
    s["x"] = P.vec(level, _random_lattice(disc, N, 10 * seed))
    if kind == "transfer":
        s["xc"], s["rc"] = P.vec(level - 1, _random_lattice(disc, N // 2, 10 * seed + 1)), P.zeros(level - 1)
        s["xf"] = P.vec(level, _random_lattice(disc, N, 10 * seed + 2))
        return s
    if kind == "apply":
        s["y"] = P.zeros(level)
        if case["op"] == "residual":
            s["b"] = P.vec(level, _random_lattice(disc, N, 10 * seed + 1))
        return s
    s["b"] = P.vec(level, _random_lattice(disc, N, 10 * seed + 1))
    if kind == "vcycle" and case["visc"]:
        for l in range(P.lmin, P.lmax + 1):
            hhg.hhg_set_viscosity(P.h, l, _nu(seed, 2 ** (l + case["macro"])).reshape(-1).contiguous())
    return s


def _smooth_omega(case):
    return {"sd": 2.34, "ml": 0.33}[case.get("schur", "sd")] if case["kind"] == "smooth" else 2.69


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "mlp_train":
        loss = hhg.hhg_mlp_train(s["t"].m, s["x"], s["y"], case["samples"], case["batch"], case["epochs"], 1e-3,
                                 s["order"])
        return {"loss": loss, "params": hhg.hhg_mlp_get_params(s["t"].m)}
    P, level = s["P"], case["level"]
    h, prec = P.h, P.prec
    gs = hhg.HHG_GS_SYM if case.get("gs") == "s" else hhg.HHG_GS_FWD
    if kind in ("fmg", "umesh_fmg"):
        hhg.hhg_fmg_solve(h, s["x"], s["bs"], s["prm"], want_stats=False)
    elif kind in ("smooth", "umesh_smooth"):
        hhg.hhg_smooth(h, level, s["x"], s["b"], case["iters"], gs, case["xi"], _smooth_omega(case), prec)
    if kind.startswith("umesh"):                        # node values in the caller's order
        hhg.hhg_vec_to_lattice(h, level, s["x"], s["out"])
        return s["out"]
    if kind in ("fmg", "smooth"):
        return s["x"]
    if kind == "vcycle":
        hhg.hhg_vcycle(h, level, s["x"], s["b"], s["prm"], prec)
        return s["x"]
    if kind == "transfer":
        hhg.hhg_restrict(h, level, s["x"], s["rc"], prec)
        hhg.hhg_prolong_add(h, level - 1, s["xc"], s["xf"], prec)
        return {"rc": s["rc"], "xf": s["xf"]}
    if case["op"] == "residual":
        hhg.hhg_residual(h, level, s["x"], s["b"], s["y"], prec)
    else:
        hhg.hhg_apply(h, level, OPS[case["op"]], s["x"], s["y"], prec)
    return s["y"]


# ------------------------------------------------------------------- work
def _dofs(case, level):
    """(velocity sites per component, pressure nodes)."""
    if case["kind"].startswith("umesh"):
        n, t = 2 ** level, np.sort(_boxes_mesh(case["boxes"])[1], axis=1)
        nv, ne, nf, nc = (len({tuple(c) for r in t.tolist() for c in itertools.combinations(r, k)}) for k in (1, 2, 3, 4))
        m = nv + ne * (n - 1) + nf * (n - 1) * (n - 2) // 2 + nc * (n - 1) * (n - 2) * (n - 3) // 6
        return m, m
    N = 2 ** (level + case["macro"])
    return ((N if case["disc"] == 1 else 2 * N) + 1) ** 3, (N + 1) ** 3


def _row_flops(case):
    """Multiply-adds x 2 per velocity site and sweep, per pressure node (both per whole row)."""
    if case["kind"].startswith("umesh"):
        return 2 * (3 * 15 + 3 * 15), 2 * (45 + 15)
    if case["disc"] == 1:
        return 2 * (3 * 7 + 3 * 14), 2 * (45 + 7)
    return 2 * (3 * (51 + 6 * 19 + 21) / 8 + 3 * 7), 2 * 3 * 65


def work(case):
    if case["kind"] == "mlp_train":
        dims = [case["n_in"], case["hidden"], case["hidden"], case["hidden"], case["n_out"]]
        par = sum(a * b + b for a, b in zip(dims, dims[1:]))
        n = case["samples"] // case["batch"] * case["batch"] * case["epochs"]
        return {"bytes": 4 * (n * (case["n_in"] + case["n_out"] + 1) + 2 * par),
                "flops": 6.0 * n * sum(a * b for a, b in zip(dims, dims[1:]))}
    w = 4 if case.get("prec") == "f32" else 8
    nv, npr = _dofs(case, case["level"])
    fv, fp = _row_flops(case)
    vec = 3 * nv + npr
    kind = case["kind"]
    if kind == "transfer":
        cv, cp = _dofs(case, case["level"] - 1)
        return {"bytes": w * (vec + 2 * (3 * cv + cp) + 2 * vec), "flops": 2.0 * 20 * vec}
    if kind == "apply":
        if case["op"] in ("A", "BT", "B", "C", "mass"):
            return {"bytes": w * 2 * vec, "flops": nv * fv + npr * fp}
        return {"bytes": w * (3 if case["op"] == "residual" else 2) * vec, "flops": nv * fv + npr * fp}
    sym = 2 if case["gs"] == "s" else 1
    it = case["xi"] * sym * nv * fv + npr * fp
    if kind in ("smooth", "umesh_smooth"):
        return {"bytes": w * 3 * vec, "flops": case["iters"] * it}
    lmin = case.get("lmin", 0)
    flops, byts = 0.0, w * 3 * vec

    def cycle(top):
        tot = 0.0
        for l in range(lmin + 1, top + 1):
            v, q = _dofs(case, l)
            n = case["pre"] + case["post"] + 2 * (top - l) * case["inc"]
            tot += n * (case["xi"] * sym * v * fv + q * fp) + v * fv + q * fp + 2.0 * 40 * (3 * v + q)
        return tot
    if kind == "vcycle":
        return {"bytes": byts, "flops": cycle(case["level"])}
    for l in range(lmin + 1, case["level"] + 1):
        flops += case["kappa"] * cycle(l)
        v, q = _dofs(case, l)
        byts += 0 if l == case["level"] else w * (3 * v + q)
    return {"bytes": byts, "flops": flops}


# ------------------------------------------------- float64 evaluation
# Finite-element reference on the definitions alone: polynomial element
# matrices, element-wise operators on lattice slices (Kuhn cube) or assembled
# sparse matrices (any tetrahedral mesh), multicolour Gauss-Seidel, linear /
# quadratic interpolation and its transpose, dense pseudo-inverse.
PERMS = list(itertools.permutations(range(3)))
GROUPS = [(0, 0, 0), (1, 0, 0), (0, 1, 0), (0, 0, 1), (1, 1, 0), (1, 0, 1), (0, 1, 1), (1, 1, 1)]  # (x, y, z) parities
DELTA = 1.0 / 12.0


def _poly_mul(p, q):
    out = {}
    for a, u in p.items():
        for b, v in q.items():
            e = tuple(i + j for i, j in zip(a, b))
            out[e] = out.get(e, 0.0) + u * v
    return out


def _poly_int(p, vol):
    """Integral over a tetrahedron of a polynomial in barycentric coordinates."""
    return sum(6 * vol * c * math.prod(math.factorial(i) for i in e) / math.factorial(sum(e) + 3) for e, c in p.items())


def _basis(order):
    """Shape functions (polynomials in the barycentric coordinates) and their nodes (sums of two vertices)."""
    u = [tuple(int(i == k) for i in range(4)) for k in range(4)]
    if order == 1:
        return [{u[k]: 1.0} for k in range(4)], [(k, k) for k in range(4)]
    add = lambda a, b: tuple(i + j for i, j in zip(a, b))  # noqa: E731
    f = [{add(u[k], u[k]): 2.0, u[k]: -1.0} for k in range(4)]
    e = list(itertools.combinations(range(4), 2))
    return f + [{add(u[i], u[j]): 4.0} for i, j in e], [(k, k) for k in range(4)] + e


def _grad(p, g):
    """Gradient (3 polynomials) given the barycentric gradients g (4, 3)."""
    out = [{}, {}, {}]
    for e, c in p.items():
        for k in range(4):
            if e[k]:
                d = tuple(x - (i == k) for i, x in enumerate(e))
                for a in range(3):
                    if g[k, a] != 0.0:
                        out[a][d] = out[a].get(d, 0.0) + c * e[k] * g[k, a]
    return out


def _elements(order):
    """Per Kuhn tetrahedron of the unit cube: vertices, velocity node positions
    (site units) and the element matrices at h = 1."""
    out = []
    for perm in PERMS:
        v = np.zeros((4, 3), int)
        for q, a in enumerate(perm):
            v[q + 1:, a] += 1
        T = np.hstack([np.ones((4, 1)), v])
        g = np.linalg.inv(T)[1:].T                       # barycentric gradients
        vol = abs(np.linalg.det(T)) / 6
        f, nodes = _basis(order)
        f1, _ = _basis(1)
        G, G1 = [_grad(p, g) for p in f], [_grad(p, g) for p in f1]
        dot = lambda a, b: sum(_poly_int(_poly_mul(x, y), vol) for x, y in zip(a, b))  # noqa: E731
        n = len(f)
        out.append(dict(
            v=v, pos=np.array([v[i] + v[j] if order == 2 else v[i] for i, j in nodes]),
            K=np.array([[dot(G[a], G[b]) for b in range(n)] for a in range(n)]),
            M=np.array([[_poly_int(_poly_mul(f[a], f[b]), vol) for b in range(n)] for a in range(n)]),
            D=np.array([[[-_poly_int(_poly_mul(f1[k], G[b][d]), vol) for b in range(n)] for k in range(4)] for d in range(3)]),
            Kp=np.array([[dot(G1[a], G1[b]) for b in range(4)] for a in range(4)]),
            Mp=np.array([[_poly_int(_poly_mul(f1[a], f1[b]), vol) for b in range(4)] for a in range(4)])))
    return out


_ELEMENTS = {}


class Lattice:
    """One level of the Kuhn cube.  Velocity (..., 3, M+1, M+1, M+1) over
    (Z, Y, X), pressure (..., N+1, N+1, N+1)."""

    def __init__(self, disc, N, schur="sd", nu=None):
        self.disc, self.N, self.h, self.M = disc, N, 1.0 / N, N if disc == 1 else 2 * N
        self.el = _ELEMENTS.setdefault(disc, _elements(disc)) if disc not in _ELEMENTS else _ELEMENTS[disc]
        self.nu = None
        if nu is not None:
            self.nu = [sum(nu[self.ps(v)] for v in e["v"]) * 0.25 for e in self.el]
        m = self.M + 1
        self.inner = torch.zeros((m, m, m), dtype=torch.bool, device=DEV)
        self.inner[1:-1, 1:-1, 1:-1] = True
        self.groups = [(0, 0, 0)] if disc == 1 else GROUPS
        self.ncol = 2 if disc == 1 else 9
        self.diag = self.scatter_v(lambda e, a, w: w * float(e["K"][a, a]) * self.h)
        self.mz = torch.zeros((N + 1,) * 3, dtype=torch.float64, device=DEV)
        for e in self.el:
            for k in range(4):
                self.mz[self.ps(e["v"][k])] += float(e["Mp"][k].sum()) * self.h ** 3
        self.dinv = 1.0 / self.mz if schur == "ml" else 1.0 / self.schur_diag()
        self.p_free = True                              # pressure fixed up to a constant

    def vs(self, pos):                                  # slices of the N^3 cubes' node at pos (x, y, z)
        st = 1 if self.disc == 1 else 2
        return (Ellipsis,) + tuple(slice(int(p), int(p) + st * (self.N - 1) + 1, st) for p in pos[::-1])

    def ps(self, v):
        return (Ellipsis,) + tuple(slice(int(p), int(p) + self.N) for p in v[::-1])

    def zeros(self, lead=()):
        return (torch.zeros(lead + (3,) + (self.M + 1,) * 3, dtype=torch.float64, device=DEV),
                torch.zeros(lead + (self.N + 1,) * 3, dtype=torch.float64, device=DEV))

    def scatter_v(self, f):
        y = torch.zeros((self.M + 1,) * 3, dtype=torch.float64, device=DEV)
        for t, e in enumerate(self.el):
            w = torch.ones((self.N,) * 3, dtype=torch.float64, device=DEV) if self.nu is None else self.nu[t]
            for a in range(len(e["pos"])):
                y[self.vs(e["pos"][a])] += f(e, a, w)
        return y

    def A(self, u, group=None, key="K", power=1):
        y = torch.zeros_like(u)
        for t, e in enumerate(self.el):
            for a, pa in enumerate(e["pos"]):
                if group is not None and self.disc == 2 and tuple(int(x) % 2 for x in pa) != group:
                    continue
                acc = None
                for b, pb in enumerate(e["pos"]):
                    w = float(e[key][a, b]) * self.h ** power
                    if abs(w) > 1e-15 * self.h ** power:
                        z = u[self.vs(pb)]
                        acc = z * w if acc is None else acc.add_(z, alpha=w)
                if acc is not None:
                    y[self.vs(pa)] += acc if self.nu is None or key != "K" else acc * self.nu[t]
        return y

    def mass(self, u, p):
        y = torch.zeros_like(p)
        for e in self.el:
            for a in range(4):
                for b in range(4):
                    y[self.ps(e["v"][a])] += float(e["Mp"][a, b]) * self.h ** 3 * p[self.ps(e["v"][b])]
        return self.A(u, None, "M", 3), y

    def BT(self, p):
        y = torch.zeros(p.shape[:-3] + (3,) + (self.M + 1,) * 3, dtype=torch.float64, device=DEV)
        for e in self.el:
            for a, pa in enumerate(e["pos"]):
                for d in range(3):
                    for k in range(4):
                        w = float(e["D"][d, k, a]) * self.h ** 2
                        if w != 0.0:
                            y.select(-4, d)[self.vs(pa)] += w * p[self.ps(e["v"][k])]
        return y

    def B(self, u):
        y = torch.zeros(u.shape[:-4] + (self.N + 1,) * 3, dtype=torch.float64, device=DEV)
        for e in self.el:
            for k in range(4):
                for a, pa in enumerate(e["pos"]):
                    for d in range(3):
                        w = float(e["D"][d, k, a]) * self.h ** 2
                        if w != 0.0:
                            y[self.ps(e["v"][k])] += w * u.select(-4, d)[self.vs(pa)]
        return y

    def C(self, p):
        y = torch.zeros_like(p)
        if self.disc == 1:
            for e in self.el:
                for a in range(4):
                    for b in range(4):
                        w = float(e["Kp"][a, b]) * DELTA * (1.0 / 6.0) ** (2.0 / 3.0) * self.h ** 3
                        y[self.ps(e["v"][a])] += w * p[self.ps(e["v"][b])]
        return y

    def schur_diag(self):
        n, st = self.N + 1, 1 if self.disc == 1 else 2
        W = {}
        for e in self.el:
            for k in range(4):
                for a, pa in enumerate(e["pos"]):
                    off = tuple(int(x) for x in pa - st * e["v"][k])
                    f = W.setdefault(off, torch.zeros((3, n, n, n), dtype=torch.float64, device=DEV))
                    for d in range(3):
                        f[d][self.ps(e["v"][k])] += float(e["D"][d, k, a]) * self.h ** 2
        ainv = torch.where(self.inner, 1.0 / self.diag, torch.zeros_like(self.diag))
        pad = torch.nn.functional.pad(ainv, (2,) * 6)
        D = torch.zeros((n, n, n), dtype=torch.float64, device=DEV)
        if self.disc == 1:
            for e in self.el:
                for k in range(4):
                    D[self.ps(e["v"][k])] += float(e["Kp"][k, k]) * DELTA * (1.0 / 6.0) ** (2.0 / 3.0) * self.h ** 3
        for off, f in W.items():
            sl = tuple(slice(2 + o, 2 + o + st * (n - 1) + 1, st) for o in off[::-1])
            D += f.square().sum(0) * pad[sl]
        return D

    def colour_mask(self, c):
        """(parity group, mask of its sites, None for all)."""
        if self.disc == 2 and c >= 2:
            return GROUPS[c - 1], None
        n = self.N + 1
        i = torch.arange(n, device=DEV)
        return (0, 0, 0), ((i[:, None, None] + i[None, :, None] + i[None, None, :]) % 2 == c)

    def sweep(self, u, rhs, order):
        """Gauss-Seidel colours of A u = rhs in place."""
        for c in order:
            g, m = self.colour_mask(c)
            st = 1 if self.disc == 1 else 2
            sl = (Ellipsis,) + tuple(slice(o, None, st) for o in g[::-1])
            r = (rhs[sl] - self.A(u, g)[sl]) / self.diag[sl]
            on = self.inner[sl] if m is None else self.inner[sl] & m
            u[sl] += torch.where(on, r, torch.zeros_like(r))

    def mask(self, u):
        return torch.where(self.inner, u, torch.zeros_like(u))

    def keep_boundary(self, u, w):
        return torch.where(self.inner, u, w)

    def interp(self, order, q):
        """Per fine class of a coarse cube (position / q): coarse offsets (site units) and weights."""
        f, nodes = _basis(order)
        for cls in itertools.product(range(q), repeat=3):
            t = np.array(cls) / q
            perm = tuple(np.argsort(-t, kind="stable"))
            v = np.zeros((4, 3), int)
            for s, a in enumerate(perm):
                v[s + 1:, a] += 1
            s = t[list(perm)]
            lam = [1 - s[0], s[0] - s[1], s[1] - s[2], s[2]]
            ws = []
            for p, (i, j) in zip(f, nodes):
                w = sum(c * math.prod(x ** k for x, k in zip(lam, e)) for e, c in p.items())
                if abs(w) > 1e-14:
                    ws.append(((v[i] + v[j]) if order == 2 else v[i], w))
            yield cls, ws

    def _transfer(self, fine, coarse, order, up):
        q, st, N = (2, 1, self.N) if order == 1 else (4, 2, self.N)   # self is the coarse level
        for cls, ws in self.interp(order, q):
            fs = (Ellipsis,) + tuple(slice(c, None, q) for c in cls[::-1])
            for o, w in ws:
                cs = (Ellipsis,) + tuple(
                    slice(int(x), int(x) + st * (N - (c > 0)) + 1, st) for x, c in zip(o[::-1], cls[::-1]))
                if up:
                    fine[fs] += w * coarse[cs]
                else:
                    coarse[cs] += w * fine[fs]

    def prolong(self, fineL, u, p):
        U, P = fineL.zeros()
        self._transfer(U, u, self.disc, True)
        self._transfer(P, p, 1, True)
        return U, P

    def restrict(self, fineL, u, p):
        U, P = self.zeros()
        self._transfer(fineL.mask(u), U, self.disc, False)
        self._transfer(p, P, 1, False)
        return self.mask(U), P

    def unknowns(self):
        return torch.nonzero(self.inner.reshape(-1)).reshape(-1)

    def pack(self, u, p):
        """The library's vector: groups of the parities, padding zero."""
        n = self.N + 1
        out = []
        for d in range(3):
            for g in self.groups:
                a = torch.zeros((n, n, n), dtype=torch.float64, device=DEV)
                s = u[d] if self.disc == 1 else u[d][tuple(slice(o, None, 2) for o in g[::-1])]
                a[tuple(slice(0, k) for k in s.shape)] = s
                out.append(a.reshape(-1))
        return torch.cat(out + [p.reshape(-1)])

    def unflatten(self, lat):
        m = (self.M + 1) ** 3
        return lat[:3 * m].reshape((3,) + (self.M + 1,) * 3).clone(), lat[3 * m:].reshape((self.N + 1,) * 3).clone()


_UMESH = {}


def _umesh(case, level):
    key = (case["boxes"], level)
    if key not in _UMESH:
        if len(_UMESH) > 8:
            _UMESH.clear()
        _UMESH[key] = Assembled(*_boxes_mesh(case["boxes"]), level)
    return _UMESH[key]


class Assembled:
    """P1-P1 level of any tetrahedral mesh by assembly.  Velocity (3, n) and
    pressure (n) over the nodes in canonical order."""

    def __init__(self, xyz, tets, level):
        n = 2 ** level
        tets = np.sort(np.asarray(tets), axis=1)
        g = np.stack(np.meshgrid(*[np.arange(n + 1)] * 3, indexing="ij"), -1).reshape(-1, 3)
        g = g[(g[:, 0] >= g[:, 1]) & (g[:, 1] >= g[:, 2])]          # lattice of a cell
        w = np.stack([n - g[:, 0], g[:, 0] - g[:, 1], g[:, 1] - g[:, 2], g[:, 2]], -1)
        local = np.full((n + 1,) * 3, -1)
        local[tuple(g.T)] = np.arange(len(g))

        def keys(tet):                                  # canonical order packed in one integer
            k = (w > 0).sum(-1).astype(np.int64) << 60
            order = np.argsort(w == 0, axis=-1, kind="stable")
            ws = np.take_along_axis(w, order, -1)
            vs = np.where(ws > 0, tet[order], 0)
            for q in range(4):
                k |= vs[..., q].astype(np.int64) << (53 - 7 * q)
                k |= ws[..., q].astype(np.int64) << (24 - 8 * q)
            return k
        lk = np.stack([keys(t) for t in tets])
        uniq, first, gid = np.unique(lk.reshape(-1), return_index=True, return_inverse=True)
        pos = np.concatenate([w @ xyz[t] for t in tets])[first] / n
        gid = torch.from_numpy(gid.reshape(lk.shape)).to(DEV)
        self.n, self.keys, self.size = n, uniq, len(uniq)
        self.dim = (uniq >> 60).astype(int)
        es, geo = [], []
        for perm in PERMS:                              # refined elements: Kuhn simplices inside the cells
            v = np.zeros((4, 3), int)
            for q, a in enumerate(perm):
                v[q + 1:, a] += 1
            c = g[:, None, :] + v[None]
            ok = ((c[..., 0] <= n) & (c[..., 0] >= c[..., 1]) & (c[..., 1] >= c[..., 2])).all(1)
            c = c[ok]
            if len(c) == 0:
                continue
            e = torch.from_numpy(local[c[..., 0], c[..., 1], c[..., 2]]).to(DEV)
            wv = np.stack([-v[:, 0], v[:, 0] - v[:, 1], v[:, 1] - v[:, 2], v[:, 2]], -1) / n
            for t, tet in enumerate(tets):              # one geometry per (cell, simplex class)
                es.append(gid[t][e])
                T = np.hstack([np.ones((4, 1)), wv @ xyz[tet]])
                geo.append((abs(np.linalg.det(T)) / 6, np.linalg.inv(T)[1:].T, len(c)))
        e = torch.cat(es)
        cnt = torch.tensor([x[2] for x in geo], device=DEV)
        rep = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(DEV).repeat_interleave(cnt, 0)  # noqa: E731
        vol, G = np.array([x[0] for x in geo]), np.stack([x[1] for x in geo])
        K = vol[:, None, None] * (G @ G.transpose(0, 2, 1))
        self.r, self.c = e.repeat_interleave(4, 1).reshape(-1), e.repeat(1, 4).reshape(-1)
        self.Amat = self.sparse(rep(K))
        self.Cmat = self.sparse(rep(DELTA * (vol ** (2 / 3))[:, None, None] * K))
        self.Mmat = self.sparse(rep(vol[:, None, None] / 20 * (np.ones((4, 4)) + np.eye(4))))
        Bd = [self.sparse(rep(np.repeat(-(vol / 4)[:, None, None] * G[:, None, :, d], 4, 1))) for d in range(3)]
        self.Bmat = Bd
        self.BTmat = [b.to_sparse_coo().t().coalesce().to_sparse_csr() for b in Bd]
        self.mz = torch.zeros(self.size, dtype=torch.float64, device=DEV)
        self.mz.index_add_(0, e.reshape(-1), rep(vol / 4).repeat_interleave(4))
        self.r = self.c = None
        coo = self.Amat.to_sparse_coo().coalesce()
        ij, v = coo.indices(), coo.values()
        self.diag = torch.zeros(self.size, dtype=torch.float64, device=DEV)
        self.diag[ij[0][ij[0] == ij[1]]] = v[ij[0] == ij[1]]
        # Dirichlet: primitives inside a face that belongs to one tetrahedron
        faces = {}
        for t in tets:
            for q in range(4):
                f = frozenset(int(x) for k, x in enumerate(t) if k != q)
                faces[f] = faces.get(f, 0) + 1
        bnd = set()
        for f, k in faces.items():
            if k == 1:
                for m in range(1, 4):
                    bnd |= {frozenset(s) for s in itertools.combinations(sorted(f), m)}
        prims, which = np.unique(uniq >> 32, return_inverse=True)
        free = np.array([frozenset(int(p >> (21 - 7 * q)) & 127 for q in range(int(p >> 28))) not in bnd for p in prims])
        self.inner = torch.from_numpy(free[which.reshape(-1)]).to(DEV)
        cc = self.Cmat.to_sparse_coo().coalesce()
        D = torch.zeros(self.size, dtype=torch.float64, device=DEV)
        on = cc.indices()[0] == cc.indices()[1]
        D[cc.indices()[0][on]] = cc.values()[on]
        ainv = torch.where(self.inner, 1.0 / self.diag, torch.zeros_like(self.diag))
        for b in Bd:
            z = b.to_sparse_coo().coalesce()
            D.index_add_(0, z.indices()[0], z.values() ** 2 * ainv[z.indices()[1]])
        self.dinv = 1.0 / D
        # colours: interface nodes greedily in canonical order, then i + j + k mod 4 in the cells
        ni = int((self.dim < 4).sum())
        i, j = ij.cpu().numpy()
        on = (i < ni) & (j < i)
        i, j = i[on], j[on]
        ptr = np.searchsorted(i, np.arange(ni + 1)).tolist()
        jl, col = j.tolist(), [0] * ni
        for q in range(ni):
            used = {col[x] for x in jl[ptr[q]:ptr[q + 1]]}
            k = 0
            while k in used:
                k += 1
            col[q] = k
        K0 = max(col) + 1
        w = np.stack([(uniq[ni:] >> (24 - 8 * q)) & 255 for q in range(4)], -1)
        col = np.concatenate([col, K0 + ((n - w[:, 0]) + (n - w[:, 0] - w[:, 1]) + w[:, 3]) % 4])
        self.ncol = K0 + 4
        rowcol = torch.from_numpy(col).to(DEV)
        self.rows = []
        for k in range(self.ncol):
            idx = torch.nonzero((rowcol == k) & self.inner).reshape(-1)
            self.rows.append((idx, self.rows_of(coo, idx)))

    def sparse(self, vals):
        s = (self.size, self.size)
        return torch.sparse_coo_tensor(torch.stack([self.r, self.c]), vals.reshape(-1), s).coalesce().to_sparse_csr()

    def rows_of(self, coo, idx):
        new = torch.full((self.size,), -1, dtype=torch.int64, device=DEV)
        new[idx] = torch.arange(len(idx), device=DEV)
        i = coo.indices()
        on = new[i[0]] >= 0
        return torch.sparse_coo_tensor(torch.stack([new[i[0][on]], i[1][on]]), coo.values()[on],
                                       (len(idx), self.size)).coalesce().to_sparse_csr()

    def zeros(self):
        return (torch.zeros((3, self.size), dtype=torch.float64, device=DEV),
                torch.zeros(self.size, dtype=torch.float64, device=DEV))

    def A(self, u):
        return (self.Amat @ u.t()).t()

    def mass(self, u, p):
        return (self.Mmat @ u.t()).t(), self.Mmat @ p

    def BT(self, p):
        return torch.stack([b @ p for b in self.BTmat])

    def B(self, u):
        return sum(b @ u[d] for d, b in enumerate(self.Bmat))

    def C(self, p):
        return self.Cmat @ p

    def sweep(self, u, rhs, order):
        for c in order:
            idx, rows = self.rows[c]
            if len(idx):
                u[:, idx] += (rhs[:, idx] - (rows @ u.t()).t()) / self.diag[idx]

    def mask(self, u):
        return torch.where(self.inner, u, torch.zeros_like(u))

    def keep_boundary(self, u, w):
        return torch.where(self.inner, u, w)

    def interp(self, fine):
        """Sparse linear interpolation (fine nodes x nodes)."""
        if getattr(self, "P", None) is None:
            w = np.stack([(fine.keys >> (24 - 8 * q)) & 255 for q in range(4)], -1)
            v = np.stack([(fine.keys >> (53 - 7 * q)) & 127 for q in range(4)], -1)
            # a fine node with lattice coordinates c (weights a) is the mean of floor(c / 2) and ceil(c / 2)
            c = np.stack([fine.n - w[:, 0], fine.n - w[:, 0] - w[:, 1], w[:, 3]], -1)
            # trailing empty weights leave the last lattice coordinates at their boundary values
            nz = fine.dim
            c[:, 2] = np.where(nz == 4, w[:, 3], 0)
            c[:, 1] = np.where(nz >= 3, fine.n - w[:, 0] - w[:, 1], 0)
            c[:, 0] = np.where(nz >= 2, fine.n - w[:, 0], 0)
            ends = []
            for d in (c // 2, (c + 1) // 2):
                a = np.stack([self.n - d[:, 0], d[:, 0] - d[:, 1], d[:, 1] - d[:, 2], d[:, 2]], -1)
                k = (a > 0).sum(-1).astype(np.int64) << 60
                order = np.argsort(a == 0, axis=-1, kind="stable")
                ws = np.take_along_axis(a, order, -1)
                vs = np.where(ws > 0, np.take_along_axis(v, order, -1), 0)
                for q in range(4):
                    k |= vs[:, q].astype(np.int64) << (53 - 7 * q)
                    k |= ws[:, q].astype(np.int64) << (24 - 8 * q)
                ends.append(np.searchsorted(self.keys, k))
            i = np.tile(np.arange(fine.size), 2)
            P = torch.sparse_coo_tensor(torch.from_numpy(np.stack([i, np.concatenate(ends)])).to(DEV),
                                        torch.full((2 * fine.size,), 0.5, dtype=torch.float64, device=DEV),
                                        (fine.size, self.size)).coalesce()
            self.P, self.R = P.to_sparse_csr(), P.t().coalesce().to_sparse_csr()
        return self.P, self.R

    def prolong(self, fine, u, p):
        P, _ = self.interp(fine)
        return (P @ u.t()).t().contiguous(), P @ p

    def restrict(self, fine, u, p):
        _, R = self.interp(fine)
        return self.mask((R @ fine.mask(u).t()).t().contiguous()), R @ p

    def unflatten(self, v):
        return v[:3 * self.size].reshape(3, self.size).clone(), v[3 * self.size:].clone()


def _operator(L, u, p):
    return L.mask(L.A(u) + L.BT(p)), L.B(u) - L.C(p)


def _mean_zero(L, p, w):
    return p - (w * p).sum() / w.sum()


def _smooth(L, u, p, fu, fp, iters, gs, xi, omega):
    for _ in range(iters):
        rhs = fu - L.BT(p)
        for _ in range(xi):
            L.sweep(u, rhs, range(L.ncol))
            if gs == "s":
                L.sweep(u, rhs, range(L.ncol - 1, -1, -1))
        p = p - omega * L.dinv * (fp - L.B(u) + L.C(p))
    return u, p


def _coarse(L, u, p, fu, fp):
    if getattr(L, "pinv", None) is None:
        free = torch.nonzero(L.inner.reshape(-1)).reshape(-1)
        nv, n = len(free), 3 * len(free) + L.mz.numel()
        K = torch.zeros((n, n), dtype=torch.float64, device=DEV)
        for c in range(n):
            eu, ep = L.zeros()
            (eu.reshape(3, -1)[c // nv].__setitem__(free[c % nv], 1.0) if c < 3 * nv
             else ep.reshape(-1).__setitem__(c - 3 * nv, 1.0))
            yu, yp = _operator(L, eu, ep)
            K[:, c] = torch.cat([yu.reshape(3, -1)[:, free].reshape(-1), yp.reshape(-1)])
        L.free, L.pinv = free, torch.from_numpy(np.linalg.pinv(K.cpu().numpy(), rcond=1e-12, hermitian=True)).to(DEV)
    yu, yp = _operator(L, u, p)
    ru, rp = fu - yu, fp - yp
    d = L.pinv @ torch.cat([ru.reshape(3, -1)[:, L.free].reshape(-1), rp.reshape(-1)])
    u, p = u.clone(), p.clone()
    u.reshape(3, -1)[:, L.free] += d[:3 * len(L.free)].reshape(3, -1)
    return u, _mean_zero(L, p + d[3 * len(L.free):].reshape(p.shape), L.mz)


def _vcycle(Ls, top, l, u, p, fu, fp, c):
    if l == 0:
        return _coarse(Ls[0], u, p, fu, fp)
    L, om = Ls[l], 1.0 / c["omega_inv"]
    u, p = _smooth(L, u, p, fu, fp, c["pre"] + (top - l) * c["inc"], c["gs"], c["xi"], om)
    yu, yp = _operator(L, u, p)
    ru, rp = Ls[l - 1].restrict(L, L.mask(fu - yu), fp - yp)
    eu, ep = _vcycle(Ls, top, l - 1, *Ls[l - 1].zeros(), ru, rp - rp.mean(), c)
    eu, ep = Ls[l - 1].prolong(L, eu, ep)
    return _smooth(L, u + L.mask(eu), p + ep, fu, fp, c["post"] + (top - l) * c["inc"], c["gs"], c["xi"], om)


def _fmg(Ls, u, fs, c):
    """u: boundary data on the finest level; fs: nodal forcing per level."""
    ws = [u]
    for l in range(len(Ls) - 1, 0, -1):                 # boundary values at the coincident nodes
        ws.insert(0, _inject(Ls[l - 1], Ls[l], ws[0]))
    bs = [(L.mask(L.mass(f, L.zeros()[1])[0]), L.zeros()[1]) for L, f in zip(Ls, fs)]
    u, p = Ls[0].zeros()
    u, p = _coarse(Ls[0], Ls[0].keep_boundary(u, ws[0]), p, *bs[0])
    for l in range(1, len(Ls)):
        u, p = Ls[l - 1].prolong(Ls[l], u, p)
        u = Ls[l].keep_boundary(u, ws[l])
        for _ in range(c["kappa"]):
            u, p = _vcycle(Ls, l, l, u, p, *bs[l], c)
            p = _mean_zero(Ls[l], p, Ls[l].mz)
    return u, p


def _inject(C, F, u):
    if isinstance(C, Lattice):
        return u[:, ::2, ::2, ::2].clone()
    k = F.keys
    w = np.stack([(k >> (24 - 8 * q)) & 255 for q in range(4)], -1)
    even = np.nonzero((w % 2 == 0).all(1))[0]
    half = k[even] & ~np.int64(0xffffffff)
    for q in range(4):
        half |= (w[even, q] // 2) << (24 - 8 * q)
    out = torch.zeros((3, C.size), dtype=torch.float64, device=DEV)
    out[:, torch.from_numpy(np.searchsorted(C.keys, half)).to(DEV)] = u[:, torch.from_numpy(even).to(DEV)]
    return out


def _exact_mlp(case, seed):
    params, x, y, order = _mlp_data(case, seed)
    P = [torch.from_numpy(p.astype(np.float32).astype(np.float64)).to(DEV) for p in params]
    m, v = [torch.zeros_like(p) for p in P], [torch.zeros_like(p) for p in P]
    x, y, order = x.double(), y.double(), torch.from_numpy(order.astype(np.int64)).to(DEV)
    n, nb, t, loss = case["samples"], case["samples"] // case["batch"], 0, 0.0
    for e in range(case["epochs"]):
        loss = 0.0
        for q in range(nb):
            idx = order[e * n + q * case["batch"]:][:case["batch"]]
            W = [p.clone().requires_grad_() for p in P]
            a = x[idx]
            for k in range(4):
                a = a @ W[2 * k].t() + W[2 * k + 1]
                a = torch.relu(a) if k < 3 else a
            l = ((a - y[idx]) ** 2).mean()
            l.backward()
            loss += float(l.detach())
            t += 1
            for k, w in enumerate(W):
                m[k] = 0.9 * m[k] + 0.1 * w.grad
                v[k] = 0.999 * v[k] + 0.001 * w.grad ** 2
                P[k] = P[k] - 1e-3 * (m[k] / (1 - 0.9 ** t)) / ((v[k] / (1 - 0.999 ** t)).sqrt() + 1e-8)
    return {"loss": loss / nb, "params": torch.cat([p.reshape(-1) for p in P]).cpu().numpy()}


def exact(case, seed):
    kind = case["kind"]
    if kind == "mlp_train":
        return _exact_mlp(case, seed)
    level = case["level"]
    rounded = (lambda v: v.float().double()) if case.get("prec") == "f32" else (lambda v: v)
    if kind.startswith("umesh"):
        if kind == "umesh_smooth":
            L = _umesh(case, level)
            u, p = L.unflatten(_u_values(L.size, seed, level, 0, 4))
            fu, fp = L.unflatten(_u_values(L.size, seed, level, 1, 4))
            u, p = _smooth(L, u, p, fu, fp, case["iters"], case["gs"], case["xi"], 1.0 / _smooth_omega(case))
        else:
            Ls = [_umesh(case, l) for l in range(level + 1)]
            u, _ = Ls[-1].unflatten(_u_values(Ls[-1].size, seed, level, 0, 3) * 0.1)
            fs = [L.unflatten(_u_values(L.size, seed, l, 1, 3))[0] for l, L in enumerate(Ls)]
            u, p = _fmg(Ls, u, fs, case)
        return torch.cat([u.reshape(-1), p])
    disc, N, schur = case["disc"], 2 ** (level + case["macro"]), case.get("schur", "sd")
    if kind == "fmg":
        ns = [2 ** (l + case["macro"]) for l in range(case["lmin"], level + 1)]
        Ls = [Lattice(disc, n) for n in ns]
        u, p = _fmg(Ls, _nodal(disc, N, seed), [_nodal(disc, n, seed + 1) * 50.0 for n in ns], case)
        return Ls[-1].pack(u, p)
    nus = case.get("visc")
    L = Lattice(disc, N, schur, _nu(seed, N) if nus else None)
    u, p = L.unflatten(rounded(_random_lattice(disc, N, 10 * seed)))
    if kind == "transfer":
        C = Lattice(disc, N // 2)
        cu, cp = C.unflatten(rounded(_random_lattice(disc, N // 2, 10 * seed + 1)))
        xu, xp = L.unflatten(rounded(_random_lattice(disc, N, 10 * seed + 2)))
        ru, rp = C.restrict(L, u, p)
        eu, ep = C.prolong(L, cu, cp)
        return {"rc": C.pack(ru, rp - rp.mean()), "xf": L.pack(xu + eu, xp + ep)}
    if kind == "apply" and case["op"] != "residual":
        op, (zu, zp) = case["op"], L.zeros()
        if op == "mass":
            return L.pack(*L.mass(u, p))
        if op == "full":
            return L.pack(*_operator(L, u, p))
        return L.pack(L.mask(L.A(u)) if op == "A" else L.mask(L.BT(p)) if op == "BT" else zu,
                      L.B(u) if op == "B" else L.C(p) if op == "C" else zp)
    fu, fp = L.unflatten(rounded(_random_lattice(disc, N, 10 * seed + 1)))
    if kind == "apply":
        yu, yp = _operator(L, u, p)
        return L.pack(L.mask(fu - yu), fp - yp)
    if kind == "smooth":
        return L.pack(*_smooth(L, u, p, fu, fp, case["iters"], case["gs"], case["xi"], 1.0 / _smooth_omega(case)))
    ns = [2 ** (l + case["macro"]) for l in range(case["lmin"], level)]
    Ls = [Lattice(disc, n, schur, _nu(seed, n) if nus else None) for n in ns] + [L]
    return L.pack(*_vcycle(Ls, len(Ls) - 1, len(Ls) - 1, u, p, fu, fp, case))
