"""Several patterns of which one alone fills the chip, so that each has a launch of its own: an odd number of
boundary dofs and columns before a pattern whose product takes the large-problem kernel, split over K and
not, against the grouped 64 x 64 schedule."""
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


def _structure(R, sizes, occs, seed):
    """Heat patterns with `sizes` boundary nodes drawn from a square mesh; every boundary node of every
    occurrence joined to one of another occurrence."""
    rng = np.random.default_rng(seed)
    pats, nodes, bn = [], [], []
    for nb in sizes:
        side = int(np.ceil(np.sqrt(1.3 * nb)))
        K = W.small_heat((side, side), (2, 1)).patterns[0].K
        b = np.sort(rng.choice(K.shape[0], nb, replace=False)).astype(np.int32)
        val = torch.from_numpy(np.ascontiguousarray(K.data)).cuda()
        p = R.pattern_factor(K.indptr, K.indices, val, b, 1, expected_kernel_dim=1)
        R.pattern_condense(p, R.FP64)
        pats.append(p)
        nodes.append(K.shape[0])
        bn.append(b)
    occ_pattern = np.repeat(np.arange(len(sizes)), occs).astype(np.int32)
    slot = np.array([(s, n) for s, p in enumerate(occ_pattern) for n in bn[p]], np.int32)
    slot = slot[rng.permutation(len(slot))]
    pair = slot[:len(slot) // 2 * 2].reshape(-1, 2, 2)
    pair = pair[pair[:, 0, 0] != pair[:, 1, 0]]
    sign = np.tile(np.array([1, -1], np.int8), (len(pair), 1))
    pb = R.problem_create(1, nodes, bn, occ_pattern, None, pair[:, :, 0], pair[:, :, 1], sign)
    return pats, pb


@pytest.mark.timeout(300)
@pytest.mark.parametrize("sizes,occs,m", [((301, 1224), (441, 33), 25),   # 10 x 7 tiles, split over K
                                          ((301, 1224), (441, 33), 26),   # an even count before it
                                          ((301, 2050), (441, 73), 25)])  # 17 x 15 tiles: K whole
def test_odd_pattern_before_the_large_kernel(R, sizes, occs, m):
    # the rule: the first pattern alone gives 256 tiles of 128 x 128, so nothing is grouped; the second gives
    # at least 192 with K in pieces of 256
    tiles = [-(-n // 128) * -(-o * m // 128) for n, o in zip(sizes, occs)]
    assert tiles[0] >= 256 and tiles[1] * min(8, sizes[1] // 256) >= 192 and sizes[0] % 2 == 1
    print(f"\n[mixed] {sizes} x {occs}, {m} columns", flush=True)
    pats, pb = _structure(R, sizes, occs, 11)
    gen = torch.Generator(device="cuda").manual_seed(m)
    X = torch.randn((pb.n_lambda, m), dtype=torch.float64, device="cuda", generator=gen)
    Y = R.feti_apply(pb, pats, X)
    N = R.feti_apply_noalloc(pb, pats, X, out=torch.empty_like(X))
    D = R.feti_precond(pb, pats, X, R.PRECOND_DIRICHLET)
    R.problem_set_schedule(pb, m, R.FP64, 64, 1024)
    G = R.feti_apply(pb, pats, X)
    E = R.feti_precond(pb, pats, X, R.PRECOND_DIRICHLET)
    torch.cuda.synchronize()
    # dot products of at most n_b terms in two orders
    tol = 4 * max(sizes) * np.finfo(float).eps
    for a, b in ((Y, G), (N, G), (D, E)):
        assert float((a - b).norm(dim=0).max()) <= tol * float(b.norm(dim=0).max())


def test_grouped_low_precision_keeps_its_pieces(R):
    """Without a schedule several small patterns share a launch, with K in as many pieces as each would have alone (8
    here: 21 x 2 tiles of 128 x 128), since FP32 sums run within a piece: the same bits as a schedule that asks
    for 8, its pieces' sums no longer."""
    pats, pb = _structure(R, (2598, 2402), (33, 33), 5)
    m = 7
    assert 1024 // (-(-2598 // 128) * -(-33 * m // 128)) >= 8
    for q in pats:
        R.pattern_condense(q, R.BF16X3)
    gen = torch.Generator(device="cuda").manual_seed(m)
    X = torch.randn((pb.n_lambda, m), dtype=torch.float64, device="cuda", generator=gen)
    Y = R.feti_apply(pb, pats, X, prec=R.BF16X3)
    R.problem_set_schedule(pb, m, R.BF16X3, 64, 4096)
    G = R.feti_apply(pb, pats, X, prec=R.BF16X3)
    torch.cuda.synchronize()
    assert torch.equal(Y, G)
