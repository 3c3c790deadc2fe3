"""The FP32 tile kernel's fused epilogues (|out|^2 after D, r - alpha (...) with r in place, both stored through
LDS), which only solves on at least 500000 sites reach, and D on a lattice between the 12-real and the
18-real limit of the tile.

The solution of the mixed solve is checked by the oracle's normal operator, and its iterations may be no more
than a tenth above the FP64 solve's.
"""
import numpy as np
import pytest

import oracle.oracle as O

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _announce():
    print("\n[gpu] test_gpu_tile_f32_solve", flush=True)


@pytest.mark.parametrize("dims", [(32, 32, 32, 16), (8, 8, 128, 62)])   # blocks of one length; of several
def test_tile_f32_fused_epilogues_in_the_mixed_solve(gpu, dims):
    import paper_1512_03487_amd as gm
    from tests.gpu_util import cached, dev, host, rel
    U, b = cached("gauge", dims, 6, kind="weak"), cached("spinor", dims, 7)
    _, s64 = gm.cg(dev(U), dev(b), "wilson", mass=1.0, tol=1e-9, sloppy="f64")
    for fmt in ("L18", "L12"):
        x, s = gm.cg(dev(U), dev(b), "wilson", mass=1.0, tol=1e-9, sloppy="f32", link_fmt=fmt)
        assert s["converged"] and s["iterations"] <= 1.1 * s64["iterations"] + 10, (fmt, s["iterations"], s64["iterations"])
        assert rel(O.normal(O.Op.wilson(1.0), U, host(x)), b) <= 1.1e-9, fmt


@pytest.mark.parametrize("fmt", ["L18", "L12"])   # share 0.75: direction-parallel, tile
def test_wilson_between_the_limits(gpu, fmt):
    import paper_1512_03487_amd as gm
    from tests.gpu_util import as_prec, cached, host, rel
    dims = (40, 24, 12, 46)
    U, psi = cached("gauge", dims, 1, kind="haar"), cached("spinor", dims, 2)
    Uk, pk, Ur, pr = as_prec(U, psi, "f32", fmt)
    for dag in (False, True):
        got, ref = host(gm.wilson(Uk, pk, 0.1, dag=dag)), O.wilson(Ur, pr, 0.1, dag)
        d = np.maximum(np.abs(got.real - ref.real), np.abs(got.imag - ref.imag)).reshape(-1, 12).max(axis=1)
        s = np.maximum(np.abs(ref.real), np.abs(ref.imag)).reshape(-1, 12).max(axis=1)
        assert rel(got, ref) <= 1e-6 and float(np.max(d / s)) <= 2.0 ** -16, (fmt, dag)
