"""GPU parity of the gauge force and the link exponential where a wavefront's run of links is cut
short: lattices whose 4 V links do not fill the last wavefront (the force, on its own and added to
the momenta by the integrators), link counts around 64, and matrices that are not in su(3).

Tolerances: 1e-13 relative for one force or exponential, 1e-12 for an integration, as for the
lattices that fill their wavefronts.
"""
import numpy as np
import pytest

from oracle import hmc as OH
from paper_1512_03487_amd import fields as F

pytestmark = pytest.mark.gpu


def _gm():
    import paper_1512_03487_amd as gm
    return gm


@pytest.fixture(scope="module", autouse=True)
def _announce():
    print("\n[gpu] test_gpu_gauge_edges", flush=True)


@pytest.mark.parametrize("dims", [(2, 2, 2, 2), (3, 3, 3, 5), (5, 3, 7, 3), (9, 2, 2, 2)])
def test_force_and_integrators_on_ragged_lattices(gpu, dims):
    from tests.gpu_util import dev, host, rel
    gm = _gm()
    U, P = F.gauge_field(dims, seed=1, kind="haar"), F.random_su3_algebra(dims, seed=7)
    assert rel(host(gm.gauge_force(dev(U), 5.7)), OH.gauge_force(U, 5.7)) <= 1e-13
    for integrator, ref in (("leapfrog", OH.leapfrog), ("omelyan", OH.omelyan), ("force_gradient", OH.force_gradient)):
        Ud, Pd = dev(U), dev(P)
        gm.md_leapfrog(Ud, Pd, 5.5, 0.05, 2, integrator=integrator)
        Ur, Pr = ref(U, P, 5.5, 0.05, 2)
        assert rel(host(Ud), Ur) <= 1e-12 and rel(host(Pd), Pr) <= 1e-12, integrator


@pytest.mark.parametrize("n", [1, 3, 63, 64, 65, 257])
def test_link_exp_counts_and_general_matrices(gpu, n):
    """exp(eps P) U for n links, P with a trace and a Hermitian part, with and without squarings."""
    import scipy.linalg as sl
    from tests.gpu_util import dev, host, rel
    rng = np.random.default_rng(n)
    U = rng.standard_normal((1, 1, 1, n, 1, 3, 3)) + 1j * rng.standard_normal((1, 1, 1, n, 1, 3, 3))
    P = 0.2 * (rng.standard_normal(U.shape) + 1j * rng.standard_normal(U.shape))
    for eps in (0.0, 0.3, -2.0):
        # api.link_exp takes whole lattices: call the library with the count itself
        import ctypes
        import torch
        from paper_1512_03487_amd import _lib
        Ud, Pd = dev(U), dev(P)
        assert _lib.load().grid_link_exp(ctypes.c_void_p(Ud.data_ptr()), ctypes.c_void_p(Pd.data_ptr()), eps, n, None) == 0
        torch.cuda.synchronize()
        ref = np.stack([sl.expm(eps * P.reshape(n, 3, 3)[k]) @ U.reshape(n, 3, 3)[k] for k in range(n)])
        assert rel(host(Ud).reshape(n, 3, 3), ref) <= 1e-13, eps
