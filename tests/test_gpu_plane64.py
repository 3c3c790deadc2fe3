"""Plane walk on 5D FP64 fields at its tile and walk edges, against the oracle.

Tolerance: FP64 1e-13 (the operator's parity tests'), per component of a site 1e-12 of its scale.
"""
import numpy as np
import pytest

import oracle.oracle as O

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _announce():
    print("\n[gpu] test_gpu_plane64", flush=True)


# One tile per plane (every face wraps onto the tile), one z plane pair, blocks of one length and of
# unequal lengths, the four Ls, several rounds of blocks; 500000 sites is where the kernel starts.
@pytest.mark.parametrize("dims,Ls", [((4, 4, 512, 16), 4), ((4, 4, 2, 2047), 8), ((8, 4, 512, 4), 8), ((16, 16, 16, 11), 12),
                                     ((16, 16, 32, 13), 8), ((8, 16, 16, 16), 16)])
@pytest.mark.parametrize("fmt", ["L18", "L12"])
def test_plane64_parity(gpu, dims, Ls, fmt):
    import paper_1512_03487_amd as gm
    from tests.gpu_util import cached, dev, host
    U, psi = cached("gauge", dims, 1, kind="haar"), cached("spinor", dims, 3, Ls=Ls)
    Uk = gm.convert_links(dev(U), "f64", fmt)
    Ur = np.asarray(U)
    for dag in (False, True):
        h = O.hop(Ur, psi, dag)
        for got, ref in ((host(gm.dhop(Uk, dev(psi), "hop", dag=dag)), h),
                         (host(gm.dwf(Uk, dev(psi), 1.8, 0.05, dag=dag)), O.dwf(Ur, psi, 1.8, 0.05, dag))):
            got, ref = got.reshape(-1, 12), ref.reshape(-1, 12)
            d = np.maximum(np.abs(got.real - ref.real), np.abs(got.imag - ref.imag)).max(axis=1)
            s = np.maximum(np.abs(ref.real), np.abs(ref.imag)).max(axis=1)
            assert np.linalg.norm(got - ref) / np.linalg.norm(ref) <= 1e-13 and float(np.max(d / s)) <= 1e-12, (dims, dag)


def test_plane64_fused_epilogues_in_the_solve(gpu):
    """|out|^2 and r - alpha (...) of the kernel inside the FP64 CG: the residual it stops at is the
    true one, and the even-odd solve (other kernels) finds the same solution."""
    import paper_1512_03487_amd as gm
    from tests.gpu_util import cached, dev
    dims = (16, 16, 16, 16)
    U, b = dev(cached("gauge", dims, 6, kind="weak")), dev(cached("spinor", dims, 7, Ls=8))
    x, st = gm.cg(U, b, "dwf", M5=1.8, mf=0.2, tol=1e-9, sloppy="f64")
    assert st["converged"] and st["true_residual"] <= 1e-9
    y = gm.dwf(U, gm.dwf(U, x, 1.8, 0.2), 1.8, 0.2, dag=True)
    assert float((y - b).norm() / b.norm()) <= 2e-9
