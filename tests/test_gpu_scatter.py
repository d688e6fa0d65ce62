"""F X of structures past the one-launch limits, at the column counts where the scatter changes its shape (1, 2, 4 and
8 columns a workgroup) and beside them, against the oracle's F: one and three dofs per node, rotated
occurrences, in the precisions whose results are scattered from column-major slabs."""
import numpy as np
import pytest

import oracle as O
import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def R():
    import paper_1208_6387_amd as R
    R.load()
    return R


def _structure(name):
    if name == "heat":
        return W.small_heat((9, 7), (8, 8))
    if name == "brick":
        return W.small_elast((3, 3, 3), (4, 4, 3))
    return W.ring_elast(24, (2, 3, 4))


@pytest.fixture(scope="module", params=["heat", "brick", "ring"])
def built(request, R):
    from paper_1208_6387_amd import structure as ST
    p = _structure(request.param)
    slots = sum(len(p.patterns[q].bnodes) for q in p.occ_pattern)
    assert slots * p.dpn > 1024          # not the one-launch form
    pats = ST.factor_patterns(p)
    ST.condense_patterns(pats, precs=(R.FP64, R.FP32, R.BF16X3))
    return p, pats, ST.create_problem(p), O.FetiOracle(p)


@pytest.mark.parametrize("m", [1, 2, 3, 4, 5, 8, 9])
def test_scatter_against_the_oracle(built, R, m):
    p, pats, pb, oracle = built
    X = np.random.default_rng(m).standard_normal((p.n_lambda, m))
    ref = oracle.F(X)
    Xd = torch.from_numpy(X).cuda()
    # FP64: the parity of S+; FP32 and bf16x3: operands to 2^-24 and 2^-16, n_b terms added in FP32
    for prec, tol in ((R.FP64, 1e-11), (R.FP32, 1e-5), (R.BF16X3, 5e-5)):
        Y = torch.full((p.n_lambda, m + 1), float("nan"), dtype=torch.float64, device="cuda")
        R.feti_apply(pb, pats, Xd, prec=prec, out=Y[:, :m])
        torch.cuda.synchronize()
        G = Y.cpu().numpy()
        assert np.linalg.norm(G[:, :m] - ref) <= tol * np.linalg.norm(ref)
        assert np.isnan(G[:, m]).all()
