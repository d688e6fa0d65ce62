"""feti_apply_noalloc where feti_apply's split of the products does not fit the fixed workspace and fewer splits are
taken: equal to feti_apply to rounding, call after call."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.timeout(300)
def test_narrow_plan_matches_feti_apply():
    import paper_1208_6387_amd as R
    from paper_1208_6387_amd import structure as ST
    R.load()
    p = W.small_elast((11, 11, 11), (3, 3, 3))
    nb, occ, m = p.patterns[0].n_b, p.n_occ, 48
    # 18 x 11 tiles of 128 x 128 with K in 5 pieces and the gathered blocks: 17.0e6 doubles, where the workspace
    # holds 16.8e6; one piece takes 5.7e6
    assert (nb, occ) == (2184, 27)
    pats = ST.factor_patterns(p)
    ST.condense_patterns(pats, (R.FP64,))
    pb = ST.create_problem(p)
    for k, cols in enumerate((m, 5, m)):
        gen = torch.Generator(device="cuda").manual_seed(k)
        X = torch.randn((p.n_lambda, cols), dtype=torch.float64, device="cuda", generator=gen)
        Y = torch.full_like(X, float("nan"))
        R.feti_apply_noalloc(pb, pats, X, out=Y)
        G = R.feti_apply(pb, pats, X)
        torch.cuda.synchronize()
        # dot products of n_b terms in two orders
        tol = 4 * nb * np.finfo(float).eps
        assert float((Y - G).norm(dim=0).max()) <= tol * float(G.norm(dim=0).max())
