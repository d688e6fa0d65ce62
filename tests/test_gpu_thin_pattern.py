"""Patterns whose interior is many bands long (the factor in band storage, its last columns included), set up
twice in a row so that the second one takes over the first one's memory, on the GPU: S against NumPy's, and the
displacements that the interior solves recover against the assembled structure's."""
import numpy as np
import pytest
import scipy.linalg as sla

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
        return W.small_heat((8, 400), (2, 1), n_rhs=2)
    return W.small_elast((3, 3, 90), (2, 1, 1), n_rhs=1)


@pytest.mark.timeout(300)
@pytest.mark.parametrize("name", ["heat", "elast"])
def test_thin_pattern_set_up_twice(R, name):
    from paper_1208_6387_amd import structure as ST
    p = _structure(name)
    pat = p.patterns[0]
    inner = np.setdiff1d(np.arange(pat.n), pat.bdofs)
    K = pat.K.toarray()
    Kii, Kib, Kbb = K[np.ix_(inner, inner)], K[np.ix_(inner, pat.bdofs)], K[np.ix_(pat.bdofs, pat.bdofs)]
    r, c = np.nonzero(Kii)
    band = int((r - c).max())
    # the band holds band + 128 + 512 rows on each side at most; the interior is more than three times that
    assert len(inner) > 3 * (band + 641)
    print(f"\n[thin] {name}: interior {len(inner)}, band {band}, boundary {len(pat.bdofs)}", flush=True)
    val = torch.from_numpy(np.ascontiguousarray(pat.K.data)).cuda()
    first = R.pattern_factor(pat.K.indptr, pat.K.indices, 1e6 * val, pat.bdofs, pat.dpn)
    first.free()
    pats = ST.factor_patterns(p)
    S = R.pattern_export(pats[0], "S").cpu().numpy()
    ref = Kbb - Kib.T @ sla.cho_solve(sla.cho_factor(Kii, lower=True), Kib)
    # backward error of a band Cholesky: a few (band + 1) eps, times the condition of K_ii
    ab = np.zeros((band + 1, len(inner)))
    for d in range(band + 1):
        ab[d, :len(inner) - d] = np.diagonal(Kii, -d)
    low = sla.eigvals_banded(ab, lower=True, select="i", select_range=(0, 0))[0]
    cond = np.abs(Kii).sum(0).max() / low
    tol = 8 * (band + 1) * np.finfo(float).eps * cond
    assert np.abs(S - ref).max() <= tol * np.abs(Kbb).max()
    ST.condense_patterns(pats, (R.FP64,))
    pb = ST.create_problem(p)
    res = R.block_krylov_solve(pb, pats, ST.loads_to_device(p), p.n_rhs, tol=1e-11, max_it=3000, method=R.ORTHODIR)
    ub, _, _, _ = O.global_solve(p)
    u = ST.split_u(p, res.u)
    assert res.stats["rel_residual"] <= 1e-11
    assert max(np.abs(a - b).max() for a, b in zip(u, ub)) <= 1e-8 * max(np.abs(b).max() for b in ub)
