"""Link gradient on its tile (4 x 4 x 2 x 2 sites) and beside it: one tile per direction (its +mu
faces wrap onto itself), several, extents it does not divide (the general kernel), short and long
sums over s. Tolerances: those of the gradient's parity tests, against the oracle.
"""
import numpy as np
import pytest

import oracle.oracle as O
from paper_1512_03487_amd import fields as F

pytestmark = pytest.mark.gpu

TOL = {"f64": 1e-13, "f32": 2e-6}


@pytest.fixture(scope="module", autouse=True)
def _announce():
    print("\n[gpu] test_gpu_grad_tile", flush=True)


@pytest.mark.parametrize("dims", [(4, 4, 2, 2), (8, 4, 6, 2), (4, 12, 2, 4), (8, 8, 3, 4), (6, 4, 4, 4)])
@pytest.mark.parametrize("Ls", [None, 1, 2, 5, 12])
@pytest.mark.parametrize("prec", ["f64", "f32"])
def test_link_grad(gpu, dims, Ls, prec):
    import paper_1512_03487_amd as gm
    from tests.gpu_util import dev, rel
    U, psi, chi = F.gauge_field(dims, seed=1), F.spinor_field(dims, seed=2, Ls=Ls), F.spinor_field(dims, seed=3, Ls=Ls)
    if prec == "f32":
        U, psi, chi = (a.astype(np.complex64) for a in (U, psi, chi))
    Ur, pr, cr = (a.astype(np.complex128) for a in (U, psi, chi))
    for dag in (False, True):
        G = O.link_grad(cr, pr, c=1.0, dag=dag)
        _, gu = gm.dhop_backward(dev(U), dev(psi), dev(chi), "hop", dag=dag, want_psi=False)
        assert rel(gu.cpu().numpy(), G) <= TOL[prec], (dims, Ls, dag)
        _, fu = gm.dhop_backward(dev(U), dev(psi), dev(chi), "hop", dag=dag, want_psi=False, force=True)
        assert rel(fu.cpu().numpy(), O.force(G, Ur)) <= 5 * TOL[prec], (dims, Ls, dag)
