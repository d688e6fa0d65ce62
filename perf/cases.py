"""Work that programs built on this library have it do, as cases that can be timed and compared.

Three kinds of call, over the sizes of the repository's own configurations and down to the smallest:

* ``setup``: factor one pattern, detect its rigid modes and condense it to the boundary flexibility
  (once per pattern of a structure, and again whenever its material changes);
* ``apply``: one product of the dual operator F (a program with an outer iteration of its own);
* ``solve``: the interface problem for a set of load cases, with the recovery of the displacements,
  on patterns and a structure that the program keeps from load set to load set.

Patterns are boxes of bilinear quads (heat) or trilinear bricks (elasticity) whose elements have
their own, random material; occurrences stand on a grid, or in the uneven assembly of thin plates on
a ring of sectors on a base block.  Solves run to 1e-11, so that what they return does not hang on
the iteration at which they stop.
"""
from functools import lru_cache

import numpy as np
import torch

import paper_1208_6387_amd as R

PREC = {"fp64": R.FP64, "fp32": R.FP32, "bf16x3": R.BF16X3}
METHOD = {"classical": R.CLASSICAL, "block_cg": R.BLOCK_CG, "orthodir": R.ORTHODIR}
PRECOND = {"none": R.PRECOND_NONE, "lumped": R.PRECOND_LUMPED, "dirichlet": R.PRECOND_DIRICHLET}
TOL = 1e-11
UNEVEN = ("24x8x2", "6x16x4", "16x16x16")  # plates, ring sectors, base block
N_SECTORS, N_PLATES = 16, 48
NOMINAL_ITERATIONS = {"none": 120, "lumped": 50, "dirichlet": 30}  # what work() charges a solve for


def listed():
    return [
        # a 2-D heat pattern, the smallest structure: launches and host work
        dict(name="setup-heat-16x16", call="setup", kind="heat", shape="16x16", prec="fp64"),
        # a ragged brick: no side a multiple of anything
        dict(name="setup-brick-7x11x5", call="setup", kind="elast", shape="7x11x5", prec="fp64"),
        # the patterns of the 64- and the 512-occurrence structures, with the copy of the mixed form
        dict(name="setup-brick-12", call="setup", kind="elast", shape="12x12x12", prec="bf16x3"),
        dict(name="setup-brick-20", call="setup", kind="elast", shape="20x20x20", prec="bf16x3"),
        # one operator product: a row of four, and the block of an outer iteration on 64 occurrences
        dict(name="apply-heat-row4", call="apply", kind="heat", shape="16x16", grid="4x1", m=3, project=False),
        dict(name="apply-64x12cube-m8", call="apply", kind="elast", shape="12x12x12", grid="4x4x4", m=8, project=True),
        # the heat row with its three permutations (full re-orthogonalisation)
        _solve("solve-heat-row4", "heat", "16x16", "4x1", 1, 3, "orthodir", "fp64"),
        # the Dirichlet preconditioner: few iterations, two products in each
        _solve("solve-27x7cube-dirichlet", "elast", "7x7x7", "3x3x3", 3, 1, "block_cg", "fp64", "dirichlet"),
        # one load case as a multivector of eight permutations, and eight load cases in the mixed form
        _solve("solve-64x12cube-8perm", "elast", "12x12x12", "4x4x4", 1, 8, "orthodir", "fp64"),
        _solve("solve-64x12cube-8rhs", "elast", "12x12x12", "4x4x4", 8, 1, "block_cg", "bf16x3"),
        # three patterns of uneven size with rotated occurrences
        _solve("solve-uneven-8perm", "elast", "uneven", "uneven", 1, 8, "orthodir", "fp64"),
        # the largest: 512 occurrences, 16 load cases, mixed form
        _solve("solve-512x20cube-16rhs", "elast", "20x20x20", "8x8x8", 16, 1, "block_cg", "bf16x3"),
    ]


def _solve(name, kind, shape, grid, n_rhs, n_perm, method, prec, precond="none"):
    case = dict(call="solve", kind=kind, shape=shape, grid=grid, n_rhs=n_rhs, n_perm=n_perm, method=method, prec=prec,
                precond=precond)
    return dict(name=name, **case) if name else case


def draw(rng):
    def log_int(lo, hi):
        return int(round(lo * (hi / lo) ** rng.random()))

    kind = rng.choice(("heat", "elast", "elast"))
    call = rng.choice(("setup", "apply", "solve", "solve"))
    if call == "setup":
        if kind == "heat":
            shape = "%dx%d" % (log_int(5, 60), log_int(5, 60))
        else:
            shape = "%dx%dx%d" % tuple(log_int(3, 18) for _ in range(3))
        return dict(call=call, kind=kind, shape=shape, prec=rng.choice(("fp64", "fp32", "bf16x3")))
    if kind == "heat":
        shape = "%dx%d" % (log_int(4, 48), log_int(4, 48))
        grid = "%dx%d" % (rng.randint(2, 8), rng.randint(1, 8))
    else:
        shape = "%dx%dx%d" % tuple(log_int(3, 13) for _ in range(3))
        grid = "%dx%dx%d" % tuple(rng.randint(2, 4) for _ in range(3))
    if call == "apply":
        return dict(call=call, kind=kind, shape=shape, grid=grid, m=log_int(1, 24), project=rng.random() < 0.5)
    n_perm = rng.choice((1, 1, 2, 5, 8))
    n_rhs = log_int(1, 16) if n_perm == 1 else rng.randint(1, 2)
    method = rng.choice(("classical", "block_cg", "orthodir")) if n_perm == 1 else "orthodir"
    return _solve(None, kind, shape, grid, n_rhs, n_perm, method, rng.choice(("fp64", "bf16x3", "fp32", "bf16x3")),
                  rng.choice(("none", "none", "lumped", "dirichlet")))


# ----------------------------------------------------------------------------- patterns

def _ints(text):
    return tuple(int(v) for v in text.split("x"))


@lru_cache(maxsize=None)
def _box(shape):
    """Lattice (node, axis), corner nodes of every element, and the stiffness of one element."""
    dim = len(shape)
    npd = tuple(s + 1 for s in shape)
    lattice = np.indices(npd[::-1]).reshape(dim, -1)[::-1].T.copy()      # x fastest
    stride = np.cumprod((1,) + npd[:-1])
    first = np.indices(shape[::-1]).reshape(dim, -1)[::-1].T @ stride
    corner = np.indices((2,) * dim).reshape(dim, -1)[::-1].T
    el = first[:, None] + corner @ stride
    h = 1.0 / max(shape)
    nen, dpn = 2 ** dim, 1 if dim == 2 else 3
    Ke = np.zeros((nen * dpn, nen * dpn))
    for g in np.indices((2,) * dim).reshape(dim, -1).T:                   # two Gauss points an axis
        x = 0.5 + (g - 0.5) / np.sqrt(3.0)
        f = np.where(corner == 1, x, 1.0 - x)
        dN = np.stack([np.where(corner[:, d] == 1, 1.0, -1.0) * np.prod(np.delete(f, d, axis=1), axis=1)
                       for d in range(dim)]) / h
        if dpn == 1:
            B, D = dN, np.eye(dim)
        else:
            lam, mu = 0.3 / (1.3 * 0.4), 0.5 / 1.3                        # E = 1, nu = 0.3
            D = np.diag([2 * mu] * 3 + [mu] * 3)
            D[:3, :3] += lam
            B = np.zeros((6, nen * 3))
            for a in range(3):
                B[a, a::3] = dN[a]
            for r, (a, b) in enumerate(((1, 2), (0, 2), (0, 1))):
                B[3 + r, a::3], B[3 + r, b::3] = dN[b], dN[a]
        Ke += B.T @ D @ B * (h / 2) ** dim
    return lattice, el, Ke, dpn, h


@lru_cache(maxsize=None)
def _csr(shape):
    """CSR structure of the assembled stiffness and the place in it of every element entry."""
    lattice, el, Ke, dpn, _ = _box(shape)
    n = len(lattice) * dpn
    dof = (el[:, :, None] * dpn + np.arange(dpn)).reshape(len(el), -1)
    key = (dof[:, :, None] * n + dof[:, None, :]).ravel()
    u, at = np.unique(key, return_inverse=True)
    rowptr = np.searchsorted(u, np.arange(n + 1, dtype=np.int64) * n).astype(np.int32)
    return rowptr, (u % n).astype(np.int32), at.ravel()


def _values(shape, rng):
    """Stiffness values with an own modulus (conductivity) in every element."""
    _, el, Ke, _, _ = _box(shape)
    rowptr, _, at = _csr(shape)
    e = np.exp(0.25 * rng.standard_normal(len(el)))
    return np.bincount(at, weights=(e[:, None] * Ke.ravel()).ravel(), minlength=rowptr[-1])


def _rigid(shape):
    """Orthonormal basis of the rigid motions (constants for heat) on the given dofs of a box."""
    lattice, _, _, dpn, h = _box(shape)
    n = len(lattice)
    if dpn == 1:
        return np.ones((n, 1))
    c = lattice * h
    Z = np.zeros((n, 3, 6))
    Z[:, (0, 1, 2), (0, 1, 2)] = 1.0
    for j, (a, b) in enumerate(((0, 1), (1, 2), (2, 0))):
        Z[:, a, 3 + j], Z[:, b, 3 + j] = -c[:, b], c[:, a]
    return Z.reshape(3 * n, 6)


# ----------------------------------------------------------------------------- structures

@lru_cache(maxsize=None)
def _structure(shape, grid, n_perm):
    if grid == "uneven":
        shapes, occ_pattern, rot, gnode, dirichlet = _uneven()
    else:
        shapes, g = (_ints(shape),), _ints(grid)
        lattice = _box(shapes[0])[0]
        place = np.indices(g[::-1]).reshape(len(g), -1)[::-1].T
        occ_pattern, rot = np.zeros(len(place), np.int32), None
        stride = np.cumprod((1,) + tuple(a * b + 1 for a, b in zip(g, shapes[0]))[:-1])
        gnode = [(lattice + p * np.array(shapes[0])) @ stride for p in place]
        # clamped where x = 0
        dirichlet = np.unique(np.concatenate([gn[lattice[:, 0] == 0] for gn, p in zip(gnode, place) if p[0] == 0]))
    # one link between neighbours in the ascending list of a shared node's occurrences, then one
    # multiplier for each clamped node, on the first occurrence that has it
    occ = np.repeat(np.arange(len(gnode)), [len(x) for x in gnode])
    node = np.concatenate([np.arange(len(x)) for x in gnode])
    g = np.concatenate(gnode)
    order = np.lexsort((occ, g))
    o, l, g = occ[order], node[order], g[order]
    a = np.nonzero(g[1:] == g[:-1])[0]
    a = a[np.lexsort((l[a], o[a + 1], o[a]))]
    first = np.concatenate([[True], g[1:] != g[:-1]])
    d = np.nonzero(first & np.isin(g, dirichlet))[0]
    d = d[np.lexsort((l[d], o[d]))]
    none = np.full(len(d), -1)
    mult_occ = np.concatenate([np.stack([o[a], o[a + 1]], 1), np.stack([o[d], none], 1)]).astype(np.int32)
    mult_node = np.concatenate([np.stack([l[a], l[a + 1]], 1), np.stack([l[d], none], 1)]).astype(np.int32)
    sign = np.where(mult_occ >= 0, np.array([1, -1]), 0).astype(np.int8)
    bnodes = []
    for p in range(len(shapes)):
        bnodes.append(np.unique(np.concatenate([mult_node[m, e] for e in range(2) for m in
                                                [(mult_occ[:, e] >= 0) & (occ_pattern[mult_occ[:, e]] == p)]])))
    # cyclic shifts among the multipliers that join the same nodes of the same patterns
    kind = np.stack([occ_pattern[mult_occ[:, 0]], np.where(mult_occ[:, 1] >= 0, occ_pattern[mult_occ[:, 1]], -1),
                     mult_node[:, 0], mult_node[:, 1]], 1)
    cls = np.unique(kind, axis=0, return_inverse=True)[1].ravel()
    by = np.lexsort((mult_occ[:, 1], mult_occ[:, 0], cls))
    size = np.bincount(cls)
    start = np.cumsum(size) - size
    pos = np.empty(len(cls), np.int64)
    pos[by] = np.arange(len(cls)) - start[cls[by]]
    perm = np.stack([by[start[cls] + (pos + k) % size[cls]] for k in range(n_perm)]).astype(np.int32)
    return dict(shapes=shapes, occ_pattern=occ_pattern, rot=rot, gnode=gnode, dirichlet=dirichlet, bnodes=bnodes,
                mult_occ=mult_occ, mult_node=mult_node, sign=sign, perm=perm, dpn=_box(shapes[0])[3])


def _uneven():
    """Sectors closed into a ring through their end faces, plates on 5 x 3 node patches of the
    sectors' outer faces, the base under the first sector; glued node by node, each in its frame."""
    shapes = tuple(_ints(t) for t in UNEVEN)
    plate, sector, base = (_box(s)[0] for s in shapes)
    npl, nse, nba = shapes

    def node(shape, ijk):
        return ijk @ np.cumprod((1,) + tuple(s + 1 for s in shape[:-1]))

    gnode, n_g = [], 0
    for s in range(N_SECTORS):
        gnode.append(n_g + np.arange(len(sector)))
        n_g += len(sector)
        if s:
            gnode[s][sector[:, 1] == 0] = gnode[s - 1][sector[:, 1] == nse[1]]
    gnode[-1][sector[:, 1] == nse[1]] = gnode[0][sector[:, 1] == 0]
    j, k = (x.ravel() for x in np.meshgrid(np.arange(5), np.arange(3), indexing="ij"))
    for q in range(N_PLATES):
        gn = n_g + np.arange(len(plate))
        n_g += len(plate)
        s, w = divmod(q, N_PLATES // N_SECTORS)
        at = node(nse, np.stack([0 * j + nse[0], 1 + 5 * w + j, 1 + k], 1))
        gn[node(npl, np.stack([0 * j, 2 + j, k], 1))] = gnode[s][at]
        gnode.append(gn)
    gn = n_g + np.arange(len(base))
    t, r = (x.ravel() for x in np.meshgrid(np.arange(nse[1] + 1), np.arange(nse[0] + 1), indexing="ij"))
    gn[node(nba, np.stack([t, r, 0 * t + nba[2]], 1))] = gnode[0][node(nse, np.stack([r, t, 0 * t], 1))]
    gnode.append(gn)
    dirichlet = gn[base[:, 2] == 0]
    occ_pattern = np.array([1] * N_SECTORS + [0] * N_PLATES + [2], np.int32)
    ang = 2 * np.pi * np.concatenate([np.arange(N_SECTORS) / N_SECTORS, np.arange(N_PLATES) / N_PLATES, [0.0]])
    rot = np.zeros((len(ang), 3, 3))
    rot[:, 0, 0] = rot[:, 1, 1] = np.cos(ang)
    rot[:, 1, 0] = np.sin(ang)
    rot[:, 0, 1] = -rot[:, 1, 0]
    rot[:, 2, 2] = 1.0
    return shapes, occ_pattern, rot, gnode, dirichlet


def _bdofs(bnodes, dpn):
    return (bnodes[:, None] * dpn + np.arange(dpn)).ravel().astype(np.int32)


def _surface(shape):
    lattice = _box(shape)[0]
    return np.nonzero(((lattice == 0) | (lattice == np.array(shape))).any(1))[0]


def _kernel_dim(dpn):
    return 1 if dpn == 1 else 6


# ----------------------------------------------------------------------------- the cases

def _structure_of(case):
    return _structure(case["shape"], case["grid"], case.get("n_perm", 1))


def _loads(st, n_rhs, seed):
    n = sum(len(g) for g in st["gnode"]) * st["dpn"]
    gen = torch.Generator(device="cuda").manual_seed(seed)
    return torch.randn(n * n_rhs, dtype=torch.float64, device="cuda", generator=gen)


def prepare(case, seed):
    rng = np.random.default_rng(seed)
    if case["call"] == "setup":
        shape = _ints(case["shape"])
        rowptr, col, _ = _csr(shape)
        dpn = _box(shape)[3]
        return dict(case=case, rowptr=rowptr, col=col, dpn=dpn, val=torch.from_numpy(_values(shape, rng)).cuda(),
                    bdofs=_bdofs(_surface(shape), dpn))
    st = _structure_of(case)
    dpn = st["dpn"]
    pb = R.problem_create(dpn, [len(_box(s)[0]) for s in st["shapes"]], st["bnodes"], st["occ_pattern"], st["rot"],
                          st["mult_occ"], st["mult_node"], st["sign"], st["perm"] if len(st["perm"]) > 1 else None)
    patterns = []
    prec = PREC[case.get("prec", "fp64")]
    for shape, bn in zip(st["shapes"], st["bnodes"]):
        rowptr, col, _ = _csr(shape)
        val = torch.from_numpy(_values(shape, rng)).cuda()
        p = R.pattern_factor(rowptr, col, val, _bdofs(bn, dpn), dpn, expected_kernel_dim=_kernel_dim(dpn))
        R.pattern_condense(p, prec)
        patterns.append(p)
    state = dict(case=case, pb=pb, patterns=patterns)
    if case["call"] == "apply":
        gen = torch.Generator(device="cuda").manual_seed(seed)
        state["X"] = torch.randn((pb.n_lambda, case["m"]), dtype=torch.float64, device="cuda", generator=gen)
        state["Y"] = torch.empty_like(state["X"])
    else:
        state["f"] = _loads(st, case["n_rhs"], seed)
        state["lam"] = torch.empty((pb.n_lambda, case["n_rhs"]), dtype=torch.float64, device="cuda")
        state["u"] = torch.empty_like(state["f"])
    return state


def run(state):
    case = state["case"]
    if case["call"] == "setup":
        p = R.pattern_factor(state["rowptr"], state["col"], state["val"], state["bdofs"], state["dpn"],
                             expected_kernel_dim=_kernel_dim(state["dpn"]))
        R.pattern_condense(p, PREC[case["prec"]])
        out = [R.pattern_export(p, "S"), R.pattern_export(p, "Splus")]
        p.free()
        return out
    if case["call"] == "apply":
        return R.feti_apply(state["pb"], state["patterns"], state["X"], project=case["project"], out=state["Y"])
    # 48 stored blocks before a restart
    R.block_krylov_solve(state["pb"], state["patterns"], state["f"], case["n_rhs"], tol=TOL, max_it=2000,
                         method=METHOD[case["method"]], prec=PREC[case["prec"]], inner_tol=1e-4, max_blocks=48,
                         lam_out=state["lam"], u_out=state["u"], precond=PRECOND[case["precond"]])
    return [state["lam"], state["u"]]


def work(case):
    def pattern(shape, n_b, dpn):
        n = len(_box(shape)[0]) * dpn
        inner = sorted(max(s - 1, 0) for s in shape)
        n_i, band = n - n_b, int(np.prod(inner[:-1])) * dpn
        return n_i, n_i * band

    if case["call"] == "setup":
        shape = _ints(case["shape"])
        dpn = _box(shape)[3]
        n_b = len(_surface(shape)) * dpn
        n_i, factor = pattern(shape, n_b, dpn)
        # band factor, one banded solve for each boundary dof, S (one triangle), inverse
        flops = factor * factor // max(n_i, 1) + 2 * n_b * factor + n_b * n_b * n_i + n_b ** 3
        return {"bytes": 8 * (len(_csr(shape)[1]) + 2 * n_b * n_b), "flops": float(flops)}
    st = _structure_of(case)
    dpn = st["dpn"]
    n_occ = np.bincount(st["occ_pattern"], minlength=len(st["shapes"]))
    n_lambda = len(st["mult_occ"]) * dpn
    m = case["m"] if case["call"] == "apply" else case["n_rhs"] * case["n_perm"]
    product = bytes_p = solves = inner = 0
    for shape, bn, c in zip(st["shapes"], st["bnodes"], n_occ):
        n_b = len(bn) * dpn
        n_i, factor = pattern(shape, n_b, dpn)
        product += 2.0 * n_b * n_b * c * m
        bytes_p += 8 * n_b * n_b
        solves += 8.0 * factor * c                   # forward and backward, for the loads and the recovery
        inner += 8 * factor
    if case["call"] == "apply":
        return {"bytes": bytes_p + 2 * 8 * n_lambda * m, "flops": float(product)}
    its, r = NOMINAL_ITERATIONS[case["precond"]], case["n_rhs"]
    loads = sum(len(g) for g in st["gnode"]) * dpn * r
    products = 2 if case["precond"] == "dirichlet" else 1
    # every iteration has to read and write its blocks: direction, product, residual, solution
    return {"bytes": bytes_p + inner + 8 * (2 * loads + its * 6 * n_lambda * m), "flops": float(its * products * product + r * solves)}


# ----------------------------------------------------------------------------- in 64 bits, plainly

def _dense(shape, val, n_b_dofs):
    """Schur complement and pseudo-inverse of a pattern's stiffness (dense, on the GPU)."""
    rowptr, col, _ = _csr(shape)
    n = len(rowptr) - 1
    K = torch.sparse_csr_tensor(torch.from_numpy(rowptr).long(), torch.from_numpy(col).long(), torch.from_numpy(val),
                                (n, n)).cuda().to_dense()
    b = torch.from_numpy(n_b_dofs).long().cuda()
    inner = torch.ones(n, dtype=torch.bool, device="cuda")
    inner[b] = False
    i = inner.nonzero().ravel()
    S = K[b][:, b]
    if len(i):
        Kib = K[i][:, b]
        Kii = K[i][:, i]
        del K
        S = S - Kib.T @ torch.cholesky_solve(Kib, torch.linalg.cholesky(Kii))
    S = 0.5 * (S + S.T)
    Z = torch.linalg.qr(torch.from_numpy(_rigid(shape)).cuda()[b])[0]
    P = Z @ Z.T
    scale = S.diagonal().mean()
    Sp = torch.cholesky_inverse(torch.linalg.cholesky(S + scale * P)) - P / scale
    return S, 0.5 * (Sp + Sp.T)


def exact(case, seed):
    rng = np.random.default_rng(seed)
    if case["call"] == "setup":
        shape = _ints(case["shape"])
        dpn = _box(shape)[3]
        return list(_dense(shape, _values(shape, rng), _bdofs(_surface(shape), dpn)))
    st = _structure_of(case)
    if sum(len(g) for g in st["gnode"]) * st["dpn"] > 1_000_000:
        return None
    vals = [_values(shape, rng) for shape in st["shapes"]]
    return _exact_apply(case, st, vals, seed) if case["call"] == "apply" else _exact_solve(case, st, vals, seed)


def _exact_apply(case, st, vals, seed):
    dpn, m = st["dpn"], case["m"]
    shape, bn = st["shapes"][0], st["bnodes"][0]
    bd = _bdofs(bn, dpn)
    Sp = _dense(shape, vals[0], bd)[1]
    n_occ, nb, n_mult = len(st["gnode"]), len(bn), len(st["mult_occ"])
    gen = torch.Generator(device="cuda").manual_seed(seed)
    X = torch.randn((n_mult * dpn, m), dtype=torch.float64, device="cuda", generator=gen)
    place = np.full(len(_box(shape)[0]), -1)
    place[bn] = np.arange(nb)
    ends = []
    for e in range(2):
        has = np.nonzero(st["mult_occ"][:, e] >= 0)[0]
        row = st["mult_occ"][has, e] * nb + place[st["mult_node"][has, e]]
        ends.append((torch.from_numpy(has).cuda(), torch.from_numpy(row).cuda(), 1.0 - 2.0 * e))

    def to_occ(v):
        w = torch.zeros((n_occ * nb, dpn, v.shape[1]), dtype=torch.float64, device="cuda")
        for has, row, sign in ends:
            w.index_add_(0, row, sign * v.view(n_mult, dpn, -1)[has])
        return w.view(n_occ, nb * dpn, -1)

    def to_mult(w):
        y = torch.zeros((n_mult, dpn, w.shape[-1]), dtype=torch.float64, device="cuda")
        for has, row, sign in ends:
            y.index_add_(0, has, sign * w.reshape(n_occ * nb, dpn, -1)[row])
        return y.view(n_mult * dpn, -1)

    w = to_occ(X)
    y = to_mult(torch.stack([Sp @ w[s] for s in range(n_occ)]))
    if not case["project"]:
        return y
    Z = torch.linalg.qr(torch.from_numpy(_rigid(shape)).cuda()[torch.from_numpy(bd).long().cuda()])[0]
    k = Z.shape[1]

    def gt(v):
        return torch.stack([Z.T @ x for x in to_occ(v)]).view(n_occ * k, -1)

    def g(a):
        return to_mult(torch.stack([Z @ x for x in a.view(n_occ, k, -1)]))

    GtG = gt(g(torch.eye(n_occ * k, dtype=torch.float64, device="cuda")))
    return y - g(torch.linalg.solve(GtG, gt(y)))


def _exact_solve(case, st, vals, seed):
    """Conjugate gradients (or dense substructures) on the assembled structure, then the multipliers from
    the nodal balances."""
    dpn, nr = st["dpn"], case["n_rhs"]
    f = _loads(st, nr, seed)
    used, inv = np.unique(np.concatenate(st["gnode"]), return_inverse=True)
    n_g = len(used)
    sizes = [len(x) for x in st["gnode"]]
    off = np.concatenate([[0], np.cumsum(sizes)])
    at = torch.from_numpy(inv.ravel()).cuda()
    rot = None if st["rot"] is None else torch.from_numpy(np.repeat(st["rot"], sizes, axis=0)).cuda()
    free = torch.ones((n_g, 1, 1), dtype=torch.float64, device="cuda")
    free[torch.from_numpy(np.searchsorted(used, st["dirichlet"])).cuda()] = 0.0
    groups = []
    for p, shape in enumerate(st["shapes"]):
        rowptr, col, _ = _csr(shape)
        n = len(rowptr) - 1
        K = torch.sparse_csr_tensor(torch.from_numpy(rowptr).long(), torch.from_numpy(col).long(),
                                    torch.from_numpy(vals[p]), (n, n)).cuda()
        occ = np.nonzero(st["occ_pattern"] == p)[0]
        nodes = torch.from_numpy(np.concatenate([np.arange(off[s], off[s + 1]) for s in occ])).cuda()
        groups.append((K, len(occ), n, nodes))

    def local(v):  # K of every occurrence on node values (node, component, case) in the occurrences' frames
        y = torch.empty_like(v)
        for K, c, n, nodes in groups:
            x = v[nodes].view(c, n, nr).permute(1, 0, 2).reshape(n, c * nr)
            y[nodes] = (K @ x).view(n, c, nr).permute(1, 0, 2).reshape(-1, dpn, nr)
        return y

    def turn(v, back):
        return v if rot is None else (rot.transpose(1, 2) if back else rot).contiguous() @ v

    def total(v):
        return torch.zeros((n_g, dpn, nr), dtype=torch.float64, device="cuda").index_add_(0, at, turn(v, False))

    def A(x):
        return free * total(local(turn(x[at].contiguous(), True)))

    fl = torch.cat([f[off[s] * dpn * nr:off[s + 1] * dpn * nr].view(nr, -1, dpn).permute(1, 2, 0)
                    for s in range(len(sizes))]).contiguous()
    rhs = free * total(fl)
    diag = torch.zeros((n_g, 1, 1), dtype=torch.float64, device="cuda")
    for p, (K, c, n, nodes) in enumerate(groups):
        rowptr, col, _ = _csr(st["shapes"][p])
        d = vals[p][col == np.repeat(np.arange(n), np.diff(rowptr))].reshape(-1, dpn).mean(1)
        diag.index_add_(0, at[nodes], torch.from_numpy(np.tile(d, c)).cuda().view(-1, 1, 1))

    def dot(a, b):
        return (a * b).sum((0, 1))

    x = torch.zeros_like(rhs)
    if rot is not None:                              # slender and ill-conditioned, but small: directly
        solve = _substructures(st, vals, inv.ravel(), off, n_g, free)
        for _ in range(3):                           # refined on the true residual
            x += solve(rhs - A(x))
    for _ in range(3 if rot is None else 0):         # restarted on the true residual
        r = rhs - A(x)
        goal = 1e-13 * dot(rhs, rhs).sqrt()
        z = r / diag
        p_, rz = z.clone(), dot(r, z)
        for it in range(4000):
            q = A(p_)
            alpha = rz / dot(p_, q).clamp_min(1e-300)
            x += alpha * p_
            r -= alpha * q
            if it % 20 == 19 and bool((dot(r, r).sqrt() <= 1e-2 * goal).all()):
                break
            z = r / diag
            rz, old = dot(r, z), rz
            p_ = z + rz / old.clamp_min(1e-300) * p_
    ul = turn(x[at].contiguous(), True)
    # what the multipliers of a node have to carry on each of its copies, in the global frame
    bal = turn(fl - local(ul), False).cpu().numpy()
    mo, mn = st["mult_occ"], st["mult_node"]
    lam = np.zeros((len(mo), dpn, nr))
    link = np.nonzero(mo[:, 1] >= 0)[0]
    for s in range(len(sizes) - 1, -1, -1):          # a chain's last copy first
        into = link[mo[link, 1] == s]
        here = off[s] + mn[into, 1]
        lam[into] = -bal[here]
        bal[off[mo[into, 0]] + mn[into, 0]] += bal[here]
    clamp = np.nonzero(mo[:, 1] < 0)[0]
    lam[clamp] = bal[off[mo[clamp, 0]] + mn[clamp, 0]]
    u = torch.cat([ul[off[s]:off[s + 1]].permute(2, 0, 1).reshape(-1) for s in range(len(sizes))])
    return [torch.from_numpy(lam.reshape(-1, nr)).cuda(), u]


def _substructures(st, vals, inv, off, n_g, free):
    """Solver of the assembled structure: dense interior factors, one dense matrix of the interface."""
    parts, dpn = [], st["dpn"]
    for p, shape in enumerate(st["shapes"]):
        rowptr, col, _ = _csr(shape)
        n = len(rowptr) - 1
        K = torch.sparse_csr_tensor(torch.from_numpy(rowptr).long(), torch.from_numpy(col).long(),
                                    torch.from_numpy(vals[p]), (n, n)).cuda().to_dense()
        b = st["bnodes"][p]
        i = np.setdiff1d(np.arange(n // dpn), b)
        bd, idf = (torch.from_numpy(_bdofs(x, dpn)).long().cuda() for x in (b, i))
        L = torch.linalg.cholesky(K[idf][:, idf])
        Kib = K[idf][:, bd]
        parts.append((b, i, L, Kib, K[bd][:, bd] - Kib.T @ torch.cholesky_solve(Kib, L)))
    touch = np.zeros(n_g, bool)
    where = []
    for s, p in enumerate(st["occ_pattern"]):
        here = inv[off[s]:off[s + 1]]
        touch[here[parts[p][0]]] = True
        where.append((here[parts[p][0]], here[parts[p][1]]))
    number = np.cumsum(touch) - 1
    keep = torch.from_numpy(np.nonzero(touch)[0]).cuda()
    size = len(keep) * dpn
    A = torch.zeros((size, size), dtype=torch.float64, device="cuda")
    dofs = []
    for s, p in enumerate(st["occ_pattern"]):
        T = torch.block_diag(*[torch.from_numpy(st["rot"][s]).cuda()] * len(parts[p][0]))
        d = torch.from_numpy(_bdofs(number[where[s][0]], dpn)).long().cuda()
        A.index_put_((d[:, None], d[None, :]), T @ parts[p][4] @ T.T, accumulate=True)
        dofs.append((T, d, torch.from_numpy(where[s][1]).cuda()))
    f = free[keep].expand(-1, dpn, 1).reshape(-1, 1)
    A = A * f * f.T + torch.diag(1.0 - f.ravel())
    LA = torch.linalg.cholesky(0.5 * (A + A.T))

    def solve(r):
        x = r.clone()
        rb = r[keep].reshape(size, -1).clone()
        for s, p in enumerate(st["occ_pattern"]):
            _, _, L, Kib, _ = parts[p]
            T, d, gi = dofs[s]
            O = torch.from_numpy(st["rot"][s]).cuda()
            y = torch.cholesky_solve((O.T @ r[gi]).reshape(len(L), -1), L)
            rb.index_add_(0, d, -(T @ (Kib.T @ y)))
        xb = f * torch.cholesky_solve(f * rb, LA)
        x[keep] = xb.view(len(keep), dpn, -1)
        for s, p in enumerate(st["occ_pattern"]):
            _, _, L, Kib, _ = parts[p]
            T, d, gi = dofs[s]
            O = torch.from_numpy(st["rot"][s]).cuda()
            y = torch.cholesky_solve((O.T @ r[gi]).reshape(len(L), -1) - Kib @ (T.T @ xb[d]), L)
            x[gi] = O @ y.view(len(gi), dpn, -1)
        return x

    return solve
