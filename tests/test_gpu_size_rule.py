"""The size rule of the flexibility products (no schedule) at the shapes where it changes kernels, against the
grouped 64 x 64 schedule on the same structure, the general path: few columns of a small pattern, the
large-problem kernel with K split and unsplit, odd boundaries, several patterns."""
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
    if name == "heat-row":               # 34 boundary dofs: few columns
        return W.small_heat((16, 16), (4, 1))
    if name == "heat-odd":               # odd boundary, several tiles
        return W.small_heat((37, 20), (3, 3))
    if name == "brick-8":                # 1,158 boundary dofs, 27 occurrences
        return W.small_elast((8, 8, 8), (3, 3, 3), n_rhs=1)
    if name == "brick-10":               # 1,806 boundary dofs
        return W.small_elast((10, 10, 10), (3, 3, 2), n_rhs=1)
    return W.uneven_three(plate=(6, 8, 2), sector=(3, 16, 4), base=16, n_sectors=4, n_perm=1)


@pytest.fixture(scope="module", params=["heat-row", "heat-odd", "brick-8", "brick-10", "uneven"])
def built(request, R):
    from paper_1208_6387_amd import structure as ST
    p = _structure(request.param)
    pats = ST.factor_patterns(p)
    ST.condense_patterns(pats, precs=(R.FP64, R.BF16X3))
    return p, pats, ST.create_problem(p)


@pytest.mark.parametrize("m", [1, 3, 8, 16, 24, 33])
@pytest.mark.parametrize("pad", [0, 3])
def test_size_rule_against_grouped(built, R, m, pad):
    p, pats, pb = built
    gen = torch.Generator(device="cuda").manual_seed(100 * m + pad)
    X = torch.randn((pb.n_lambda, m + pad), dtype=torch.float64, device="cuda", generator=gen)[:, :m]
    Y = torch.full((pb.n_lambda, m + pad), float("nan"), dtype=torch.float64, device="cuda")[:, :m]
    R.feti_apply(pb, pats, X, out=Y)
    R.problem_set_schedule(pb, m, R.FP64, 64, 1024)
    G = R.feti_apply(pb, pats, X.contiguous())
    R.problem_set_schedule(pb, m, R.FP64, 0)
    N = R.feti_apply_noalloc(pb, pats, X, out=torch.empty_like(G))
    torch.cuda.synchronize()
    # dot products of at most n_b terms in two orders
    nb = max(q.n_b for q in pats)
    tol = 4 * nb ** 0.5 * np.finfo(float).eps * float(G.norm(dim=0).max())
    assert float((Y - G).norm(dim=0).max()) <= tol * max(1.0, nb ** 0.5)
    assert float((N - G).norm(dim=0).max()) <= tol * max(1.0, nb ** 0.5)


@pytest.mark.parametrize("m", [1, 8, 17])
def test_low_precision_size_rule(built, R, m):
    p, pats, pb = built
    gen = torch.Generator(device="cuda").manual_seed(m)
    X = torch.randn((pb.n_lambda, m), dtype=torch.float64, device="cuda", generator=gen)
    Y = R.feti_apply(pb, pats, X, prec=R.BF16X3)
    G = R.feti_apply(pb, pats, X)
    torch.cuda.synchronize()
    # operands to 2^-16 each, against the size of the terms (S+ w cancels little on random blocks)
    assert float((Y - G).norm()) <= 5e-5 * float(G.norm())


@pytest.mark.parametrize("m", [1, 5, 16, 40])
def test_projected_product(built, R, m):
    """Q^T F X: its coarse solve in blocks of 16 columns, G^T of the result zero to rounding."""
    p, pats, pb = built
    gen = torch.Generator(device="cuda").manual_seed(7 * m)
    X = torch.randn((pb.n_lambda, m), dtype=torch.float64, device="cuda", generator=gen)
    Y = R.feti_apply(pb, pats, X, project=True)
    Z = R.feti_precond(pb, pats, Y.clone(), R.PRECOND_NONE, project=True)
    torch.cuda.synchronize()
    assert float((Z - Y).norm()) <= 1e-9 * float(R.feti_apply(pb, pats, X).norm())
