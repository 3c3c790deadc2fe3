"""exp(eps P) U where P is no su(3) element: matrices that contract or grow by many orders of magnitude,
each link to the relative accuracy that its own size allows.

Reference: P = a + A with A in su(3), exp(P) = exp(a) exp(A), exp(A) from the eigenvectors of the
Hermitian -i A. Tolerance: the scaled exponential is off by a few units in the last place, taken as
8 x 2^-53, and every squaring doubles that: 8 x 2^-53 x 2^k per link, 2^k the least power above
2 |eps P|.
"""
import numpy as np
import pytest

from paper_1512_03487_amd import fields as F

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _announce():
    print("\n[gpu] test_gpu_link_exp_general", flush=True)


@pytest.mark.parametrize("eps", [1.0, -0.5])
@pytest.mark.parametrize("a", [-40.0, -10.0, -1.0, -0.25, 0.0, 0.25, 3.0, 40.0])
def test_link_exp_that_contracts_or_grows(gpu, a, eps):
    import paper_1512_03487_amd as gm
    from tests.gpu_util import dev, host
    dims = (3, 5, 2, 2)
    U, A = F.gauge_field(dims, seed=1, kind="haar"), F.random_su3_algebra(dims, seed=6)
    P = A + a * np.eye(3)
    Ud = dev(U)
    gm.link_exp(Ud, dev(P), eps)
    w, v = np.linalg.eigh(-1j * eps * A)
    ref = np.exp(eps * a) * (np.einsum("...ij,...j,...kj->...ik", v, np.exp(1j * w), v.conj()) @ U)
    got, ref = host(Ud).reshape(-1, 9), ref.reshape(-1, 9)
    err = np.linalg.norm(got - ref, axis=1) / np.linalg.norm(ref, axis=1)
    k = np.maximum(0, np.ceil(np.log2(2 * abs(eps) * np.linalg.norm(P.reshape(-1, 9), axis=1))))
    # the reference's own phases: a rounding of w each
    tol = (8 * 2.0 ** k + 4 * (1 + np.abs(w).max())) * 2.0 ** -53
    assert np.all(err <= tol), float(np.max(err / tol))
