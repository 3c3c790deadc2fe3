"""Plane walk on checkerboard fields (Ls = 16, FP32 and FP16 storage) at its tile and walk edges.

Tolerances: those of the checkerboard operator's parity tests (FP32 1e-6 against the oracle on the
FP32-rounded inputs, FP16 storage 2e-3); per component of a site, 2^-16 and 2^-10 of its scale.
"""
import numpy as np
import pytest

from oracle import eo
from paper_1512_03487_amd import fields as F

pytestmark = pytest.mark.gpu

TOL = {"f32": 1e-6, "f16s": 2e-3}
SITE_TOL = {"f32": 2.0 ** -16, "f16s": 2.0 ** -10}


@pytest.fixture(scope="module", autouse=True)
def _announce():
    print("\n[gpu] test_gpu_plane_cb", flush=True)


def _site_err(got, ref) -> float:
    got, ref = got.reshape(-1, 12), ref.reshape(-1, 12)
    d = np.maximum(np.abs(got.real - ref.real), np.abs(got.imag - ref.imag)).max(axis=1)
    s = np.maximum(np.abs(ref.real), np.abs(ref.imag)).max(axis=1)
    return float(np.max(d / s))


# 8 x 4 with one tile per plane (every halo wraps); 4 x 8: the 2 x 8 tile; walks of one slice, of two
# and of unequal length (34 slices in 12 blocks); Lz = 2 (z + 1 = z - 1); Lt = 2.
DIMS = [(8, 4, 2, 256), (4, 8, 2, 256), (16, 8, 16, 14), (12, 8, 12, 22), (8, 4, 512, 2), (16, 8, 16, 34)]


@pytest.mark.parametrize("dims", DIMS)
@pytest.mark.parametrize("prec,fmt", [("f32", "L18"), ("f32", "L12"), ("f16s", "L18"), ("f16s", "L12")])
def test_plane_cb_parity(gpu, dims, prec, fmt):
    import paper_1512_03487_amd as gm
    from tests.gpu_util import as_prec, cached, host, rel
    vol = int(np.prod(dims))
    if prec == "f16s":   # FP16 storage takes the kernel from 400000 sites on
        dims = dims[:2] + ((dims[2], 2 * dims[3]) if vol * 16 < 400000 else dims[2:])
    assert int(np.prod(dims)) * 16 >= 200000
    U = cached("gauge", dims, 1, kind="haar")
    psi, y = cached("spinor", dims, 3, Ls=16), cached("spinor", dims, 4, Ls=16)
    for p in (0, 1):
        Uk, pk, Ur, pr = as_prec(U, eo.pick(psi, 1 - p), prec, fmt)
        _, yk, _, yr = as_prec(U, eo.pick(y, p), prec, fmt)
        dag = (p == 1) != (fmt == "L12")
        h = eo.hop_cb(Ur, pr, p, dag)
        got = host(gm.dhop_cb(Uk, pk, p, "hop", beta=0.75, dag=dag))
        assert rel(got, 0.75 * h) <= TOL[prec] and _site_err(got, 0.75 * h) <= SITE_TOL[prec], (dims, p, dag, "hop")
        ref = eo.m5(yr, 1.8, 0.05, dag) - 0.25 * h
        got = host(gm.dhop_cb(Uk, pk, p, "dwf", y=yk, beta=-0.25, M5=1.8, mf=0.05, dag=dag))
        assert rel(got, ref) <= TOL[prec] and _site_err(got, ref) <= SITE_TOL[prec], (dims, p, dag, "dwf")


@pytest.mark.parametrize("prec", ["f32", "f16s"])
@pytest.mark.parametrize("beta", [0.0, 1e-9, 1e9])
def test_plane_cb_beta_far_from_one_keeps_the_column_walk(gpu, prec, beta):
    """beta = 0 and extreme beta take the general kernel: the same bounds hold."""
    import paper_1512_03487_amd as gm
    from tests.gpu_util import as_prec, cached, host, rel
    dims = (8, 8, 16, 28)
    U = cached("gauge", dims, 1, kind="haar")
    psi, y = cached("spinor", dims, 3, Ls=16), cached("spinor", dims, 4, Ls=16)
    Uk, pk, Ur, pr = as_prec(U, eo.pick(psi, 1), prec)
    _, yk, _, yr = as_prec(U, eo.pick(y, 0), prec)
    ref = eo.m5(yr, 1.8, 0.05, False) + beta * eo.hop_cb(Ur, pr, 0, False)
    got = host(gm.dhop_cb(Uk, pk, 0, "dwf", y=yk, beta=beta, M5=1.8, mf=0.05))
    assert rel(got, ref) <= TOL[prec]


@pytest.mark.parametrize("kind,kw", [("dwf", dict(M5=1.8, mf=0.1)), ("mobius", dict(M5=1.8, mf=0.1, b5=1.5, c5=0.5)),
                                     ("mobius", dict(M5=1.8, mf=0.1, b5=1.0, c5=0.0))])
@pytest.mark.parametrize("sloppy,dims", [("f32", (8, 8, 8, 26)), ("f16s", (4, 8, 28, 28))])
def test_plane_cb_in_the_even_odd_solve(gpu, kind, kw, sloppy, dims):
    """The kinds with (d - S)^-1 and B run only inside solve_eo. The mixed solve corrects by FP64
    residuals, so a wrong sloppy operator shows in the iteration count: it may need no more than a
    quarter (FP32: a tenth) above what the FP64 operators need, and the solution is the same."""
    import torch
    import paper_1512_03487_amd as gm
    from tests.gpu_util import cached, dev
    U, b = dev(cached("gauge", dims, 6, kind="weak")), dev(cached("spinor", dims, 7, Ls=16))
    x64, s64 = gm.solve_eo(U, b, kind, tol=1e-9, sloppy="f64", **kw)
    x, s = gm.solve_eo(U, b, kind, tol=1e-9, sloppy=sloppy, **kw)
    it64, it = s64["iterations"], s["iterations"]
    assert it <= it64 * (1.1 if sloppy == "f32" else 1.25) + 10, (it, it64)
    assert float((x - x64).norm() / x64.norm()) <= 1e-6
