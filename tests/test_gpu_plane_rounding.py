"""Rounding error of the FP32 plane walks: no larger than the column walk's, which the same call takes on
smaller lattices (its eight hops are summed before the larger diagonal part joins them).

The relative error of a whole field of independent Gaussian values does not depend on the lattice: over
the smaller field's 1.5 million components its statistical spread is 1e-3, and 2 % are allowed. An order
that rounds every hop at the size of the diagonal part is 9 to 75 % off.
"""
import pytest

pytestmark = pytest.mark.gpu

SMALL, LARGE = (8, 8, 8, 8), (16, 16, 8, 12)   # x Ls = 16: 65536 sites (column walk) and 393216


@pytest.fixture(scope="module", autouse=True)
def _announce():
    print("\n[gpu] test_gpu_plane_rounding", flush=True)


@pytest.mark.parametrize("b5,c5", [(1.5, 0.5), (2.0, 1.0)])
@pytest.mark.parametrize("dag", [False, True])
def test_mobius_rounding(gpu, dag, b5, c5):
    import paper_1512_03487_amd as gm
    from oracle import mobius as MB
    from tests.gpu_util import as_prec, cached, host, rel
    err = {}
    for dims in (SMALL, LARGE):
        U, psi = cached("gauge", dims, 1, kind="haar"), cached("spinor", dims, 3, Ls=16)
        Uk, pk, Ur, pr = as_prec(U, psi, "f32")
        err[dims] = rel(host(gm.mobius(Uk, pk, 1.8, 0.3, b5, c5, dag=dag)), MB.mobius(Ur, pr, 1.8, 0.3, b5, c5, dag))
    assert err[LARGE] <= 1.02 * err[SMALL], err


@pytest.mark.parametrize("beta", [-0.25, -2.0 ** -8, 0.7])
@pytest.mark.parametrize("dag", [False, True])
def test_checkerboard_rounding(gpu, dag, beta):
    import paper_1512_03487_amd as gm
    from oracle import eo
    from tests.gpu_util import as_prec, cached, host, rel
    err = {}
    for dims in (SMALL, LARGE):
        U, psi, y = cached("gauge", dims, 1, kind="haar"), cached("spinor", dims, 3, Ls=16), cached("spinor", dims, 4, Ls=16)
        Uk, pk, Ur, pr = as_prec(U, eo.pick(psi, 1), "f32")
        _, yk, _, yr = as_prec(U, eo.pick(y, 0), "f32")
        got = host(gm.dhop_cb(Uk, pk, 0, "dwf", y=yk, beta=beta, M5=1.8, mf=0.05, dag=dag))
        err[dims] = rel(got, eo.m5(yr, 1.8, 0.05, dag) + beta * eo.hop_cb(Ur, pr, 0, dag))
    assert err[LARGE] <= 1.02 * err[SMALL], err


@pytest.mark.parametrize("prec,rel_tol,site_tol", [("f32", 1e-6, 2.0 ** -16), ("f16s", 2e-3, 2.0 ** -10)])
@pytest.mark.parametrize("beta", [0.0, 2.0 ** -21, -2.0 ** -19, 2.0 ** 19, -2.0 ** 21, 1e9])
def test_checkerboard_of_any_beta(gpu, prec, rel_tol, site_tol, beta):
    """No beta divides anything: 0 and factors far from 1, on fields the plane walk takes in both storages
    (638976 full-lattice sites), to the bounds of its parity tests."""
    import numpy as np
    import paper_1512_03487_amd as gm
    from oracle import eo
    from tests.gpu_util import as_prec, cached, host, rel
    dims = (8, 8, 24, 26)
    U, psi, y = cached("gauge", dims, 1, kind="haar"), cached("spinor", dims, 3, Ls=16), cached("spinor", dims, 4, Ls=16)
    Uk, pk, Ur, pr = as_prec(U, eo.pick(psi, 1), prec)
    _, yk, _, yr = as_prec(U, eo.pick(y, 0), prec)
    ref = eo.m5(yr, 1.8, 0.05, False) + beta * eo.hop_cb(Ur, pr, 0, False)
    got = host(gm.dhop_cb(Uk, pk, 0, "dwf", y=yk, beta=beta, M5=1.8, mf=0.05))
    g, r = got.reshape(-1, 12), ref.reshape(-1, 12)
    d = np.maximum(np.abs(g.real - r.real), np.abs(g.imag - r.imag)).max(axis=1)
    s = np.maximum(np.abs(r.real), np.abs(r.imag)).max(axis=1)
    assert rel(got, ref) <= rel_tol and float(np.max(d / s)) <= site_tol, (prec, beta)
