"""Rounding of the setup and of the dense solve, against LAPACK's on the same data, both measured from references
whose residuals are taken in long double: S+ of whole bricks, and rpf_dposv up to a condition of 1e11."""
import numpy as np
import pytest
import scipy.linalg as sl
import scipy.sparse as sp

from workloads import mesh as WM

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
LD = np.longdouble


@pytest.fixture(scope="module")
def R():
    import paper_1208_6387_amd as R
    R.load()
    return R


def _norm(x):
    return float(np.linalg.norm(x.astype(float)))


def _rigid(c):
    """Orthonormal rigid motions of nodes at c, in long double."""
    Z = np.zeros((len(c), 3, 6), LD)
    Z[:, (0, 1, 2), (0, 1, 2)] = 1
    for j, (a, b) in enumerate(((0, 1), (1, 2), (2, 0))):
        Z[:, a, 3 + j], Z[:, b, 3 + j] = -c[:, b], c[:, a]
    Q = Z.reshape(-1, 6)
    for _ in range(3):
        for j in range(6):
            for i in range(j):
                Q[:, j] -= Q[:, i] * (Q[:, i] @ Q[:, j])
            Q[:, j] /= np.sqrt(Q[:, j] @ Q[:, j])
    return Q


def _brick(shape, rng):
    """Stiffness of a box of bricks with an own modulus in each, node coordinates, which nodes are outside."""
    mesh = WM.GridMesh(shape, [x / max(shape) for x in shape])
    el = mesh.elements()
    Ke = WM.hex_elasticity(*mesh.h)
    dof = (el[:, :, None] * 3 + np.arange(3)).reshape(len(el), -1)
    val = (np.exp(0.25 * rng.standard_normal(len(el)))[:, None] * Ke.ravel()).ravel()
    n = 3 * mesh.n_nodes
    K = sp.coo_matrix((val, (np.repeat(dof, 24, axis=1).ravel(), np.tile(dof, (1, 24)).ravel())), shape=(n, n)).tocsr()
    K.sum_duplicates()
    K = 0.5 * (K + K.T).tocsr()
    K.sort_indices()
    on = np.zeros(mesh.n_nodes, bool)
    on[mesh.surface_nodes()] = True
    return K, mesh.coords, on


def test_pseudo_inverse_rounds_no_more_than_lapack(R):
    """S+ on random self-equilibrated tractions, for two bricks with two materials each."""
    gpu = lapack = 0.0
    rng = np.random.default_rng(0)
    for shape in ((7, 7, 7), (9, 8, 8), (7, 7, 7), (9, 8, 8)):
        K, c, on = _brick(shape, rng)
        b = np.nonzero(np.repeat(on, 3))[0].astype(np.int32)
        i = np.nonzero(~np.repeat(on, 3))[0]
        n = K.shape[0]
        p = R.pattern_factor(K.indptr, K.indices, torch.from_numpy(np.ascontiguousarray(K.data)).cuda(), b, 3,
                             expected_kernel_dim=6)
        R.pattern_condense(p)
        Sp = R.pattern_export(p, "Splus").cpu().numpy()
        p.free()
        Kd = K.toarray()
        Q = _rigid(c.astype(LD))
        Qb = _rigid(c[on].astype(LD))
        # plain LAPACK: S, then the inverse of S + Z Z^T by Cholesky
        S = Kd[np.ix_(b, b)] - Kd[np.ix_(b, i)] @ sl.cho_solve(sl.cho_factor(Kd[np.ix_(i, i)], lower=True), Kd[np.ix_(i, b)])
        Z = Qb.astype(float)
        P, info = sl.lapack.dpotri(sl.cholesky(0.5 * (S + S.T) + Z @ Z.T, lower=True), lower=1)
        assert info == 0
        P = np.tril(P) + np.tril(P, -1).T - Z @ Z.T
        # reference: the Neumann solution, refined, its trace orthogonal to the rigid motions
        y = rng.standard_normal((len(b), 6)).astype(LD)
        y -= Qb @ (Qb.T @ y)
        f = np.zeros((n, 6), LD)
        f[b] = y
        sc = K.diagonal().mean()
        M = sl.cho_factor(Kd + sc * (Q @ Q.T).astype(float), lower=True)
        val, u = K.data.astype(LD)[:, None], np.zeros((n, 6), LD)
        for _ in range(8):
            Ku = np.add.reduceat(val * u[K.indices], K.indptr[:-1], axis=0)
            u += sl.cho_solve(M, (f - Ku - LD(sc) * (Q @ (Q.T @ u))).astype(float))
        ub = u[b] - Qb @ (Qb.T @ u[b])
        e = [_norm(T.astype(LD) @ y - ub) / _norm(ub) for T in (Sp, P)]
        print(f"\n[rounding] {shape}: {e[0]:.2e}, LAPACK {e[1]:.2e}", flush=True)
        gpu += e[0]
        lapack += e[1]
    assert gpu <= 1.05 * lapack


@pytest.mark.parametrize("cond", [1e2, 1e6, 1e11])
@pytest.mark.parametrize("n", [700, 1100])
def test_dense_solve_residual(R, n, cond):
    """The residual of rpf_dposv stays within twice the substitution's (LAPACK), whatever the condition, for few
    and for many columns."""
    rng = np.random.default_rng(n)
    Qm = np.linalg.qr(rng.standard_normal((n, n)))[0]
    A = (Qm * np.exp(rng.permutation(np.linspace(0, -np.log(cond), n)))) @ Qm.T
    A = 0.5 * (A + A.T)
    B = rng.standard_normal((n, 120))
    ref = sl.cho_solve(sl.cho_factor(A, lower=True), B)

    def residual(X):
        r = np.concatenate([A[k:k + 256].astype(LD) @ X.astype(LD) for k in range(0, n, 256)]) - B[:, :X.shape[1]]
        return _norm(r) / np.linalg.norm(X)

    for cols in (7, 120):
        Ad = torch.from_numpy(np.ascontiguousarray(A.T)).cuda().T
        Bd = torch.from_numpy(np.ascontiguousarray(B[:, :cols].T)).cuda().T
        R.dposv(Ad, Bd)
        torch.cuda.synchronize()
        assert residual(Bd.cpu().numpy()) <= 2 * residual(ref[:, :cols])


def test_more_columns_than_the_second_buffer(R):
    """Columns are taken in turn past the second buffer's bound (2^22 of them for three rows)."""
    n, cols = 3, (1 << 22) + 5
    A = np.array([[4.0, 1.0, 0.5], [1.0, 3.0, 0.25], [0.5, 0.25, 2.0]])
    B = torch.randn((cols, n), dtype=torch.float64, device="cuda", generator=torch.Generator(device="cuda").manual_seed(1))
    X = B.clone()
    R.dposv(torch.from_numpy(A.copy()).cuda().T, X.T)
    r = X @ torch.from_numpy(A).cuda() - B
    assert float(r.abs().max()) <= 32 * np.finfo(float).eps * float(X.abs().max()) * 5.5
