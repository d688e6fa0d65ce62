"""Rounding of the one-launch forms of small structures (F X, and its projection) against the general path's on the
same data: both measured from the products in long double."""
import numpy as np
import pytest

import oracle as O
import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
LD = np.longdouble


@pytest.fixture(scope="module")
def R():
    import paper_1208_6387_amd as R
    R.load()
    return R


def _structure(name):
    if name == "heat-row":
        return W.small_heat((16, 16), (4, 1))
    if name == "brick-2":
        return W.small_elast((2, 2, 2), (2, 2, 2))
    return W.ring_elast(4, (1, 2, 1))


@pytest.mark.parametrize("name", ["heat-row", "brick-2", "ring"])
def test_one_launch_rounds_no_more_than_the_general_path(R, name):
    from paper_1208_6387_amd import structure as ST
    p = _structure(name)
    m = 64
    pats = ST.factor_patterns(p)
    ST.condense_patterns(pats, (R.FP64,))
    pb = ST.create_problem(p)
    Sp = [R.pattern_export(q, "Splus").cpu().numpy().astype(LD) for q in pats]
    A = [a.toarray().astype(LD) for a in O.FetiOracle(p).A]
    X = np.random.default_rng(1).standard_normal((p.n_lambda, m))
    ref = sum(A[s] @ (Sp[q] @ (A[s].T @ X.astype(LD))) for s, q in enumerate(p.occ_pattern))
    Xd = torch.from_numpy(X).cuda()
    one = R.feti_apply(pb, pats, Xd).cpu().numpy()
    R.problem_set_schedule(pb, m, R.FP64, 64, 1024)     # a schedule names the general path
    general = R.feti_apply(pb, pats, Xd).cpu().numpy()
    e = [float(np.linalg.norm((y - ref).astype(float))) for y in (one, general)]
    print(f"\n[rounding] {name}: one launch {e[0]:.3e}, general {e[1]:.3e}", flush=True)
    assert e[0] <= 1.1 * e[1]
