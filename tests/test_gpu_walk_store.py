"""FP32 stores of the column walks, which leave a wavefront's records as one run of lines: fields whose
columns end inside a wavefront or a block, full and checkerboard, plain and Moebius.

Tolerance: FP32 1e-6 against the oracle on the FP32-rounded inputs (the operators' parity tests'), per
component of a site 2^-16 of its scale, so that a misplaced record cannot pass; the guard records
after the output stay as they were.
"""
import numpy as np
import pytest

import oracle.oracle as O
from oracle import eo
from oracle import mobius as MB
from paper_1512_03487_amd import fields as F

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _announce():
    print("\n[gpu] test_gpu_walk_store", flush=True)


def _check(got, ref, tag):
    got, ref = got.reshape(-1, 12), ref.reshape(-1, 12)
    d = np.maximum(np.abs(got.real - ref.real), np.abs(got.imag - ref.imag)).max(axis=1)
    s = np.maximum(np.abs(ref.real), np.abs(ref.imag)).max(axis=1)
    assert np.linalg.norm(got - ref) / np.linalg.norm(ref) <= 1e-6 and float(np.max(d / s)) <= 2.0 ** -16, tag


def _guarded(shape):
    import torch
    n = int(np.prod(shape))
    buf = torch.full((n + 3072,), 7.0, dtype=torch.complex64, device="cuda:0")
    return buf, buf[:n].view(shape)


@pytest.mark.parametrize("dims,Ls", [((2, 2, 2, 2), 2), ((2, 3, 5, 4), 5), ((6, 2, 2, 3), 6), ((4, 6, 2, 4), 8),
                                     ((3, 5, 3, 2), 24), ((2, 2, 3, 4), 16)])
def test_walk_stores(gpu, dims, Ls):
    import paper_1512_03487_amd as gm
    from tests.gpu_util import as_prec
    U, psi = F.gauge_field(dims, seed=1, kind="haar"), F.spinor_field(dims, seed=2, Ls=Ls)
    Uk, pk, Ur, pr = as_prec(U, psi, "f32")
    buf, out = _guarded(tuple(pk.shape))
    for dag in (False, True):
        gm.dwf(Uk, pk, 1.8, 0.05, dag=dag, out=out)
        _check(out.cpu().numpy(), O.dwf(Ur, pr, 1.8, 0.05, dag), (dims, Ls, dag))
        if 64 % Ls == 0:
            gm.mobius(Uk, pk, 1.8, 0.05, 1.5, 0.5, dag=dag, out=out)
            _check(out.cpu().numpy(), MB.mobius(Ur, pr, 1.8, 0.05, 1.5, 0.5, dag), (dims, Ls, dag, "mobius"))
    assert bool((buf[-3072:] == 7.0).all())


@pytest.mark.parametrize("dims,Ls", [((2, 2, 2, 2), 2), ((6, 2, 2, 4), 5), ((4, 6, 2, 4), 8), ((2, 4, 6, 2), 24)])
def test_walk_cb_stores(gpu, dims, Ls):
    import paper_1512_03487_amd as gm
    from tests.gpu_util import as_prec
    U, psi, y = F.gauge_field(dims, seed=1, kind="haar"), F.spinor_field(dims, seed=2, Ls=Ls), F.spinor_field(dims, seed=3, Ls=Ls)
    for p in (0, 1):
        Uk, pk, Ur, pr = as_prec(U, eo.pick(psi, 1 - p), "f32")
        _, yk, _, yr = as_prec(U, eo.pick(y, p), "f32")
        buf, out = _guarded(tuple(pk.shape))
        for dag in (False, True):
            h = eo.hop_cb(Ur, pr, p, dag)
            gm.dhop_cb(Uk, pk, p, "dwf", y=yk, beta=-0.25, M5=1.8, mf=0.05, dag=dag, out=out)
            _check(out.cpu().numpy(), eo.m5(yr, 1.8, 0.05, dag) - 0.25 * h, (dims, Ls, p, dag))
        assert bool((buf[-3072:] == 7.0).all())
