"""F X of small structures in one launch, against the grouped products of a schedule on the same structure: one to
three dofs per node, rotated occurrences, several patterns, single endpoints, strided blocks and the block in place."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def R():
    import paper_1208_6387_amd as R
    R.load()
    return R


def _structure(name):
    if name == "heat-row":
        return W.small_heat((16, 16), (4, 1))
    if name == "heat-2cube":             # 64 occurrences of 8 boundary nodes
        return W.small_heat((2, 2), (8, 8))
    if name == "heat-65":                # one occurrence more than the single launch takes
        return W.small_heat((2, 2), (13, 5))
    if name == "brick-2":                # 78 boundary dofs, 624 rows
        return W.small_elast((2, 2, 2), (2, 2, 2))
    if name == "brick-3":                # more boundary dofs than the single launch takes
        return W.small_elast((3, 3, 3), (2, 2, 1))
    if name == "mirror-row":             # two patterns
        return W.mirror_row_heat(4)
    return W.ring_elast(3, (2, 2, 2))


@pytest.fixture(scope="module", params=["heat-row", "heat-2cube", "heat-65", "brick-2", "brick-3", "mirror-row",
                                        "ring-elast"])
def built(request, R):
    from paper_1208_6387_amd import structure as ST
    p = _structure(request.param)
    pats = ST.factor_patterns(p)
    ST.condense_patterns(pats, precs=(R.FP64,))
    return p, pats, ST.create_problem(p)


@pytest.mark.parametrize("m", [1, 2, 7, 32, 33, 130])
@pytest.mark.parametrize("project", [False, True])
def test_small_apply(built, R, m, project):
    p, pats, pb = built
    gen = torch.Generator(device="cuda").manual_seed(m)
    X = torch.randn((pb.n_lambda, m + 2), dtype=torch.float64, device="cuda", generator=gen)[:, 1:m + 1]
    Y = torch.full((pb.n_lambda, m + 3), float("nan"), dtype=torch.float64, device="cuda")
    R.feti_apply(pb, pats, X, project=project, out=Y[:, :m])
    N = R.feti_apply_noalloc(pb, pats, X, out=torch.empty_like(X))
    Z = X.clone()
    R.feti_apply(pb, pats, Z, project=project, out=Z)      # in place
    # one buffer, two strides: overlapping rows take the general path
    buf = torch.zeros(pb.n_lambda * (m + 2), dtype=torch.float64, device="cuda")
    A = buf.as_strided((pb.n_lambda, m), (m + 2, 1))
    B = buf.as_strided((pb.n_lambda, m), (m, 1))
    A.copy_(X)
    R.feti_apply(pb, pats, A, project=project, out=B)
    R.problem_set_schedule(pb, m, R.FP64, 64, 1024)
    F = R.feti_apply(pb, pats, X.contiguous())
    G = R.feti_apply(pb, pats, X.contiguous(), project=True) if project else F
    R.problem_set_schedule(pb, m, R.FP64, 0)
    torch.cuda.synchronize()
    assert bool(torch.isnan(Y[:, m:]).all())
    # dot products of at most n_b terms in two orders
    nb = max(q.n_b for q in pats)
    tol = 4 * nb * np.finfo(float).eps * float(F.norm(dim=0).max())
    assert float((Y[:, :m] - G).norm(dim=0).max()) <= tol
    assert float((N - F).norm(dim=0).max()) <= tol
    assert float((Z - G).norm(dim=0).max()) <= tol
    assert float((B - G).norm(dim=0).max()) <= tol


@pytest.mark.parametrize("m", [1, 8, 33, 130])
def test_small_projection(built, R, m):
    """Q X by itself and behind the product, against the oracle's G on both sides of the single launch's limits."""
    import oracle as O
    p, pats, pb = built
    o = O.FetiOracle(p)
    gen = torch.Generator(device="cuda").manual_seed(1000 + m)
    X = torch.randn((pb.n_lambda, m + 1), dtype=torch.float64, device="cuda", generator=gen)[:, :m]
    P = R.feti_precond(pb, pats, X, R.PRECOND_NONE, project=True)
    F = R.feti_apply(pb, pats, X)
    Y = R.feti_apply(pb, pats, X, project=True)
    torch.cuda.synchronize()
    # the explicit inverse of G^T G, and kernels of two factorisations
    cond = np.linalg.cond(o.GtG) if o.GtG.size else 1.0
    tol = 1024 * np.finfo(float).eps * max(cond, 100.0)
    for got, of in ((P, X), (Y, F)):
        ref = of.cpu().numpy()
        want = o.Q(ref)
        assert np.linalg.norm(got.cpu().numpy() - want) <= tol * np.linalg.norm(ref)
