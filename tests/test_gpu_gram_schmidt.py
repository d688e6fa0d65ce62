"""Kernels of the floating strips whose boundary sizes lie at the edges of the orthonormalisation's row counts: the
detected kernel is the constant vector, of unit length, whatever kernel took the detection block."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n_b", [6, 8, 10, 510, 512, 514, 1022, 1024, 1026, 2046, 2048, 2050, 4094, 4096, 4098])
def test_kernel_of_a_strip(n_b):
    import paper_1208_6387_amd as R
    R.load()
    from paper_1208_6387_amd import structure as ST
    p = W.small_heat((2, n_b // 2 - 1), (3, 1))
    pat = ST.factor_patterns(p)[0]
    assert pat.n_b == n_b
    Z = R.pattern_export(pat, "Z")
    torch.cuda.synchronize()
    Z = Z.reshape(-1).cpu().numpy()
    assert Z.shape == (n_b,)
    eps = np.finfo(float).eps
    assert abs(np.linalg.norm(Z) - 1.0) <= 16 * eps
    # entries of the Schur complement to a few eps, its next eigenvalue is about 10 / n_b^2 of its norm
    assert np.linalg.norm(np.abs(Z) - n_b ** -0.5) <= 16 * eps * n_b ** 2
