"""The FP64 plane walk's fused epilogues inside the CG, against operators that are not the kernel itself: the
oracle's normal operator on the solution, and the even-odd solve, which runs the checkerboard kernels.
"""
import pytest

import oracle.oracle as O

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _announce():
    print("\n[gpu] test_gpu_plane64_solve", flush=True)


@pytest.mark.parametrize("dims,Ls", [((16, 16, 16, 16), 8), ((4, 4, 512, 16), 4)])
def test_plane64_solution(gpu, dims, Ls):
    import paper_1512_03487_amd as gm
    from tests.gpu_util import cached, dev, host, rel
    U, b = cached("gauge", dims, 6, kind="weak"), cached("spinor", dims, 7, Ls=Ls)
    x, st = gm.cg(dev(U), dev(b), "dwf", M5=1.8, mf=0.2, tol=1e-9, sloppy="f64")
    assert st["converged"]
    assert rel(O.normal(O.Op.dwf(Ls, 1.8, 0.2), U, host(x)), b) <= 1.1e-9
    # M^dagger M x = b in two even-odd solves: M^dagger z = b has no entry point, so M x = z with z = M x formed
    # by the oracle
    z = O.dwf(U, host(x), 1.8, 0.2)
    xe, _ = gm.solve_eo(dev(U), dev(z), "dwf", tol=1e-11, sloppy="f64", M5=1.8, mf=0.2)
    assert rel(host(xe), host(x)) <= 1e-8
