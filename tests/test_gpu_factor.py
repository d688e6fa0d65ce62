"""The blocked Cholesky factor and its triangular solves at the edges of their tiles (16), diagonal blocks
(128) and panels, against NumPy, on the GPU: through rpf_dposv."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def R():
    import paper_1208_6387_amd as R
    R.load()
    return R


def cm(a, pad=0):
    """Host array -> column-major device tensor whose leading dimension has `pad` spare rows (NaN)."""
    t = torch.full((a.shape[1], a.shape[0] + pad), float("nan"), dtype=torch.float64)
    t[:, :a.shape[0]] = torch.from_numpy(np.ascontiguousarray(a.T))
    return t.cuda().T[:a.shape[0]]


@pytest.mark.parametrize("cols", [1, 5, 17, 70])
@pytest.mark.parametrize("n,pad", [(15, 0), (16, 1), (17, 0), (127, 0), (128, 0), (129, 1), (143, 0), (144, 3), (255, 1),
                                   (256, 0), (257, 0), (385, 0), (512, 0), (513, 2), (1100, 0), (1537, 0)])
def test_factor_and_solve(R, n, pad, cols):
    rng = np.random.default_rng(1000 * n + cols)
    X = rng.standard_normal((n, n))
    A = X @ X.T / n + np.eye(n)
    B = rng.standard_normal((n, cols))
    Ad, Bd = cm(A, pad), cm(B, pad)
    R.dposv(Ad, Bd)
    torch.cuda.synchronize()
    G = Ad.cpu().numpy()
    # condition number below 6: errors of a few n eps
    tol = 8 * n * np.finfo(float).eps
    assert np.abs(np.tril(G) - np.linalg.cholesky(A)).max() <= tol * 2
    assert np.array_equal(np.triu(G, 1), np.triu(A, 1))
    assert np.abs(Bd.cpu().numpy() - np.linalg.solve(A, B)).max() <= tol * np.abs(B).max()


@pytest.mark.parametrize("scale", [2.0 ** -900, 2.0 ** 900])
@pytest.mark.parametrize("n", [5, 40, 200])
def test_factor_far_from_one(R, n, scale):
    """Powers of four times a matrix: the factor is that power of two times the matrix's, to the bit."""
    rng = np.random.default_rng(n)
    X = rng.standard_normal((n, n))
    A = X @ X.T / n + np.eye(n)
    A1, A2 = cm(A), cm(A * scale)
    R.dposv(A1)
    R.dposv(A2)
    torch.cuda.synchronize()
    assert np.array_equal(np.tril(A1.cpu().numpy()) * np.sqrt(scale), np.tril(A2.cpu().numpy()))


@pytest.mark.parametrize("n,bad", [(40, 0), (40, 39), (300, 130), (300, 299)])
def test_factor_refuses_a_pivot(R, n, bad):
    d = np.ones(n)
    d[bad] = -1.0
    with pytest.raises(R.RpfError, match="ENOTSPD"):
        R.dposv(cm(np.diag(d)))
