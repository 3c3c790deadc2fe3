"""Tiled walk of 4D FP16-storage and FP32 fields at its tile and walk edges: one tile per direction (every face
wraps onto the tile's own far side), several, walks of one slice and of unequal length.

Tolerances: FP16 storage 2e-3, FP32 1e-6 (the parity tests'), per component of a site 2^-10 and 2^-16
of its scale.
"""
import numpy as np
import pytest

import oracle.oracle as O

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _announce():
    print("\n[gpu] test_gpu_tile", flush=True)


@pytest.mark.parametrize("dims", [(8, 8, 4, 2), (8, 16, 12, 7), (24, 8, 8, 5), (8, 8, 4, 300),
                                  (16, 32, 32, 13)])
@pytest.mark.parametrize("fmt", ["L18", "L12"])
def test_tile_parity(gpu, dims, fmt):
    import paper_1512_03487_amd as gm
    from tests.gpu_util import as_prec, cached, host, rel
    U, psi = cached("gauge", dims, 1, kind="haar"), cached("spinor", dims, 2)
    Uk, pk, Ur, pr = as_prec(U, psi, "f16s", fmt)
    for dag in (False, True):
        for got, ref in ((host(gm.dhop(Uk, pk, "hop", dag=dag)), O.hop(Ur, pr, dag)),
                         (host(gm.wilson(Uk, pk, 0.1, dag=dag)), O.wilson(Ur, pr, 0.1, dag))):
            d = np.maximum(np.abs(got.real - ref.real), np.abs(got.imag - ref.imag)).reshape(-1, 12).max(axis=1)
            s = np.maximum(np.abs(ref.real), np.abs(ref.imag)).reshape(-1, 12).max(axis=1)
            assert rel(got, ref) <= 2e-3 and float(np.max(d / s)) <= 2.0 ** -10, (dims, fmt, dag)


# FP32 takes the kernel from 500000 sites on: one round of even blocks; z extent 2 (both z faces the
# same plane); x and y extent 8 (faces of the tile itself) and walks of unequal length.
@pytest.mark.parametrize("dims", [(32, 32, 32, 16), (64, 64, 2, 64), (8, 8, 128, 62)])
@pytest.mark.parametrize("fmt", ["L18", "L12"])
def test_tile_parity_f32(gpu, dims, fmt):
    import paper_1512_03487_amd as gm
    from tests.gpu_util import as_prec, cached, host, rel
    U, psi = cached("gauge", dims, 1, kind="haar"), cached("spinor", dims, 2)
    Uk, pk, Ur, pr = as_prec(U, psi, "f32", fmt)
    for dag in (False, True):
        got = host(gm.wilson(Uk, pk, 0.1, dag=dag))
        ref = O.wilson(Ur, pr, 0.1, dag)
        d = np.maximum(np.abs(got.real - ref.real), np.abs(got.imag - ref.imag)).reshape(-1, 12).max(axis=1)
        s = np.maximum(np.abs(ref.real), np.abs(ref.imag)).reshape(-1, 12).max(axis=1)
        assert rel(got, ref) <= 1e-6 and float(np.max(d / s)) <= 2.0 ** -16, (dims, fmt, dag)


@pytest.mark.parametrize("dims", [(8, 8, 4, 6), (16, 8, 8, 14)])
def test_tile_fused_epilogues_in_the_mixed_solve(gpu, dims):
    """The kernel's |out|^2 and r - alpha (...) epilogues, inside the FP16-storage CG: the same
    solution, and no more than a quarter more iterations than with FP64 operators."""
    import paper_1512_03487_amd as gm
    from tests.gpu_util import cached, dev
    U, b = dev(cached("gauge", dims, 6, kind="weak")), dev(cached("spinor", dims, 7))
    x64, s64 = gm.cg(U, b, "wilson", mass=0.3, tol=1e-9, sloppy="f64")
    for fmt in ("L18", "L12"):
        x, s = gm.cg(U, b, "wilson", mass=0.3, tol=1e-9, sloppy="f16s", link_fmt=fmt)
        assert s["iterations"] <= 1.25 * s64["iterations"] + 10, (s["iterations"], s64["iterations"])
        assert float((x - x64).norm() / x64.norm()) <= 1e-6
