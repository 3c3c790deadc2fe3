"""GPU parity of the plane walk (5D FP32 / FP16-storage fields with Ls = 8, 12 or 16, at least 160000
and 300000 sites; FP32 with Ls = 20 or 24, at least 400000; on lattices whose x and y extents its
tiles divide) at the sizes where it can go wrong: one tile per direction (every face wraps), odd numbers of planes and slices, tiles in the
interior, walks of several slices and of one, and lattices on either side of its limits.

Tolerances as for the other schedules (tests/test_gpu_dhop.py): FP32 1e-6 and FP16 storage 2e-3 over
the field, and per component 2^-16 / 2^-10 of the site's largest component.
"""
import numpy as np
import pytest

import oracle.oracle as O
from paper_1512_03487_amd import fields as F

pytestmark = pytest.mark.gpu

TOL = {"f32": 1e-6, "f16s": 2e-3}
SITE_TOL = {"f32": 2.0 ** -16, "f16s": 2.0 ** -10}


def _gm():
    import paper_1512_03487_amd as gm
    return gm


@pytest.fixture(scope="module", autouse=True)
def _announce():
    print("\n[gpu] test_gpu_plane", flush=True)


def _check(got, ref, prec, what):
    from tests.gpu_util import rel
    assert rel(got, ref) <= TOL[prec], what
    g, r = got.reshape(-1, 12), ref.reshape(-1, 12)
    d = np.maximum(np.abs(g.real - r.real), np.abs(g.imag - r.imag)).max(axis=1)
    s = np.maximum(np.abs(r.real), np.abs(r.imag)).max(axis=1)
    assert float(np.max(d / s)) <= SITE_TOL[prec], what


# (Lx, Ly, Lz, Lt), Ls: 4 x 4 tiles for Ls = 12, 16; 8 x 4 and 4 x 8 for Ls = 8. The first of a pair
# stays below the FP16-storage limit (column walk there); Lx = 6 and, in FP16 storage, Ls = 20 and 24 are the
# column walk's.
SHAPES = [((4, 4, 41, 20), 16), ((4, 4, 79, 16), 16), ((8, 4, 71, 11), 8), ((8, 4, 121, 10), 8), ((4, 8, 131, 9), 8),
          ((12, 8, 23, 12), 12), ((8, 16, 17, 18), 8), ((16, 12, 8, 13), 16), ((6, 4, 41, 26), 12), ((4, 4, 32, 32), 20),
          ((4, 4, 41, 31), 20), ((4, 8, 41, 13), 24), ((12, 8, 16, 11), 24)]


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("prec,fmt", [("f32", "L18"), ("f32", "L12"), ("f16s", "L18"), ("f16s", "L12")])
def test_plane_parity(gpu, shape, prec, fmt):
    from tests.gpu_util import as_prec, cached, host
    gm = _gm()
    dims, Ls = shape
    U, psi = cached("gauge", dims, 1, kind="haar"), cached("spinor", dims, 3, Ls=Ls)
    Uk, pk, Ur, pr = as_prec(U, psi, prec, fmt)
    for dag in (False, True):
        _check(host(gm.dwf(Uk, pk, 1.8, 0.3, dag=dag)), O.dwf(Ur, pr, 1.8, 0.3, dag), prec, ("dwf", dag))
        _check(host(gm.dhop(Uk, pk, "hop", dag=dag)), O.hop(Ur, pr, dag), prec, ("hop", dag))


@pytest.mark.parametrize("sloppy", ["f32", "f16s"])
@pytest.mark.parametrize("shape", [((8, 12, 26, 12), 12), ((8, 4, 121, 10), 8), ((4, 8, 41, 13), 24)])
def test_plane_fused_epilogues(gpu, sloppy, shape):
    """Mixed-precision CG (the norm and r-update epilogues) to a small FP64 residual."""
    from tests.gpu_util import dev, host, rel
    gm = _gm()
    dims, Ls = shape
    U = F.gauge_field(dims, seed=1, kind="haar")
    b = F.spinor_field(dims, seed=3, Ls=Ls)
    x, st = gm.cg(dev(U), dev(b), kind="dwf", M5=1.8, mf=0.1, tol=1e-10, sloppy=sloppy, check_every=4)
    assert st["converged"]
    back = O.normal(O.Op.dwf(Ls, 1.8, 0.1), U, host(x))
    assert rel(back, b) <= 1.1e-10


@pytest.mark.parametrize("shape", [((4, 4, 41, 20), 16), ((4, 4, 79, 16), 16), ((16, 12, 8, 13), 16), ((16, 16, 16, 6), 16)])
@pytest.mark.parametrize("prec,fmt", [("f32", "L18"), ("f32", "L12"), ("f16s", "L18"), ("f16s", "L12")])
def test_plane_mobius_parity(gpu, shape, prec, fmt):
    """The Moebius operator on the plane walk (Ls = 16: a fifth-dimension column per 16-lane row)."""
    from oracle import mobius as MB
    from tests.gpu_util import as_prec, cached, host
    gm = _gm()
    dims, Ls = shape
    U, psi = cached("gauge", dims, 1, kind="haar"), cached("spinor", dims, 3, Ls=Ls)
    Uk, pk, Ur, pr = as_prec(U, psi, prec, fmt)
    for dag in (False, True):
        got = host(gm.mobius(Uk, pk, 1.8, 0.3, 1.5, 0.5, dag=dag))
        _check(got, MB.mobius(Ur, pr, 1.8, 0.3, 1.5, 0.5, dag), prec, dag)


@pytest.mark.parametrize("sloppy", ["f32", "f16s"])
def test_plane_mobius_fused_epilogues(gpu, sloppy):
    from oracle import mobius as MB
    from tests.gpu_util import dev, host, rel
    gm = _gm()
    dims, Ls = (16, 8, 16, 10), 16
    U = F.gauge_field(dims, seed=1, kind="haar")
    b = F.spinor_field(dims, seed=3, Ls=Ls)
    x, st = gm.cg(dev(U), dev(b), kind="mobius", M5=1.8, mf=0.1, b5=1.5, c5=0.5, tol=1e-10, sloppy=sloppy, check_every=4)
    assert st["converged"]
    assert rel(MB.normal(U, host(x), 1.8, 0.1, 1.5, 0.5), b) <= 1.1e-10
