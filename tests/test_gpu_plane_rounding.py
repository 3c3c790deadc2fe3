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
