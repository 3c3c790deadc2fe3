"""4D FP16-storage fields on the column walks: D with 12-real links (the same-step walk) on ragged lattices and
on ones the tile divides but leaves to it (2 to 2.83 slices of a block per CU), at both ends of that range,
with the fused epilogues inside the mixed solve.

Tolerances as for the tiled walk: 2e-3 over the field, per component 2^-10 of the site's largest.
"""
import numpy as np
import pytest

import oracle.oracle as O

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _announce():
    print("\n[gpu] test_gpu_walk_4d", flush=True)


# blocks x Lt / 256: 2.0 (the tile), 2.06, 2.81, 2.86 (the tile); extents that divide nothing; the smallest
@pytest.mark.parametrize("dims", [(16, 16, 16, 32), (16, 16, 16, 33), (24, 24, 20, 16), (8, 16, 24, 61), (21, 5, 6, 7), (3, 2, 2, 2),
                                  (2, 2, 2, 2)])
@pytest.mark.parametrize("fmt", ["L18", "L12"])
def test_walk_4d_parity(gpu, dims, fmt):
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


@pytest.mark.parametrize("dims", [(6, 6, 6, 10), (16, 16, 16, 33)])
def test_walk_4d_fused_epilogues_in_the_mixed_solve(gpu, dims):
    import paper_1512_03487_amd as gm
    from tests.gpu_util import cached, dev, host, rel
    U, b = cached("gauge", dims, 6, kind="weak"), cached("spinor", dims, 7)
    x64, s64 = gm.cg(dev(U), dev(b), "wilson", mass=0.3, tol=1e-9, sloppy="f64")
    x, s = gm.cg(dev(U), dev(b), "wilson", mass=0.3, tol=1e-9, sloppy="f16s", link_fmt="L12")
    assert s["iterations"] <= 1.25 * s64["iterations"] + 10, (s["iterations"], s64["iterations"])
    assert rel(O.normal(O.Op.wilson(0.3), U, host(x)), b) <= 1.1e-9


# blocks x Lt / 256: 4.0 (the tile), 4.06, 4.92, 5.06 (the tile), and 4.69 in slices of 15360 sites (the tile)
@pytest.mark.parametrize("dims", [(16, 16, 32, 32), (16, 16, 16, 65), (8, 16, 40, 63), (16, 16, 16, 81), (24, 40, 16, 20)])
@pytest.mark.parametrize("fmt", ["L18", "L12"])
def test_walk_4d_parity_four_to_five_slices(gpu, dims, fmt):
    test_walk_4d_parity(gpu, dims, fmt)


def test_walk_4d_fused_epilogues_four_to_five_slices(gpu):
    test_walk_4d_fused_epilogues_in_the_mixed_solve(gpu, (8, 16, 40, 63))
