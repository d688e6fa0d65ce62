"""The coarse solve of wide blocks and large coarse spaces: Q X at the widths where the product changes its kernel,
against the same columns taken eight at a time."""
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def R():
    import paper_1208_6387_amd as R
    R.load()
    return R


@pytest.mark.timeout(300)
@pytest.mark.parametrize("grid,widths", [((8, 8, 5), (32, 33)),          # n_G = 1,920: two kernels by width
                                         ((8, 8, 8), (16, 17, 33, 70)),  # 3,072
                                         ((10, 9, 8), (3, 16, 40))])     # 4,320: split over K at every width
def test_wide_projection(R, grid, widths):
    from paper_1208_6387_amd import structure as ST
    p = W.small_elast((2, 2, 2), grid)
    print(f"\n[coarse] {grid}: {6 * p.n_occ} coarse unknowns", flush=True)
    pats = ST.factor_patterns(p)
    ST.condense_patterns(pats, (R.FP64,))
    pb = ST.create_problem(p)
    for m in widths:
        gen = torch.Generator(device="cuda").manual_seed(m)
        X = torch.randn((pb.n_lambda, m), dtype=torch.float64, device="cuda", generator=gen)
        Y = R.feti_precond(pb, pats, X, R.PRECOND_NONE, project=True)
        parts = [R.feti_precond(pb, pats, X[:, j:j + 8].contiguous(), R.PRECOND_NONE, project=True)
                 for j in range(0, m, 8)]
        torch.cuda.synchronize()
        # sums of n_G products in two orders: sqrt(n_G) eps times the condition of G^T G (a few thousand)
        assert float((Y - torch.cat(parts, 1)).norm()) <= 1e-10 * float(X.norm())
        Z = R.feti_precond(pb, pats, Y, R.PRECOND_NONE, project=True)   # a projector
        torch.cuda.synchronize()
        assert float((Z - Y).norm()) <= 1e-10 * float(X.norm())
