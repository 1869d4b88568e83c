"""Kernels at the edges of their ranges: first and last tile, remainders, and
both sides of every size rule, against numpy / scipy in FP64."""
import numpy as np
import pytest
import scipy.linalg

from tests.gpu_util import requires_gpu

pytestmark = [pytest.mark.gpu, requires_gpu]


@pytest.fixture(scope="module")
def handle():
    import paper_2105_00578_amd as sx
    return sx.Handle(0)


@pytest.mark.parametrize("w,m", [(1, 1), (2, 1), (2, 2), (7, 7), (8, 3), (22, 7), (23, 7),
                                 (31, 9), (32, 9), (33, 11), (47, 16)])
def test_rayleigh_ritz_orders(handle, w, m):
    """Odd and even orders, one / two / five blocks per thread.  The pencil's
    condition is that of Z^T Z for a 300 x w normal Z (below 10), so a
    backward-stable solve has errors of some w * 2^-53 ||GA||, w^2 with the
    norms' bounds: 1e-12 ||GA|| leaves a factor above 4."""
    from paper_2105_00578_amd import _lib
    rng = np.random.default_rng(100 + w)
    Z = rng.standard_normal((300, w))
    GB = Z.T @ Z
    A = rng.standard_normal((w, w))
    GA = A + A.T
    Y, th, kept, bd = _lib.rayleigh_ritz(handle, m, GA, GB)
    assert bd == 0 and kept == w
    ref = scipy.linalg.eigh(GA, GB, eigvals_only=True)[:m]
    scale = np.linalg.norm(GA) / 300
    assert np.allclose(th, ref, rtol=0, atol=1e-12 * scale)
    assert np.allclose(Y.T @ GB @ Y, np.eye(m), atol=1e-12)
    assert np.allclose(GA @ Y, GB @ Y @ np.diag(th), atol=1e-12 * np.linalg.norm(GA))
