"""How a Bloch operator's application rounds: on the FE rows the finite-element part m^-1/2 sum(Y) and the
coupling H^co Z^O are each summed by itself and added once, so that the products of many enrichment functions do
not round at the size of the finite-element part.  Then H(u + v) for a block u without enrichment rows and a
block v without FE rows is the rounded sum of H u and H v, to the bit."""
import numpy as np
import pytest

from paper_2010_09701_amd import workloads as wl

pytestmark = pytest.mark.gpu

K = np.array([0.21, -0.37, 0.13])


@pytest.mark.parametrize("uform", [False, True])
@pytest.mark.parametrize("dt", ["complex64", "complex128"])
@pytest.mark.parametrize("nv", [1, 7, 24])
def test_parts_are_added_once(dt, nv, uform):
    import torch
    from paper_2010_09701_amd import oefe
    op = oefe.Operator(wl.diamond8(nc=4, p=3).with_k(K), uform=uform)
    X = torch.from_numpy(wl.start_block(op.n_tot, nv, 6, complex_=True)).to(getattr(torch, dt)).cuda()
    u, v = X.clone(), X.clone()
    u[op.n_fe:] = 0
    v[:op.n_fe] = 0
    v *= 1e-2
    Y, Yu, Yv = (oefe.ham_apply(op, B)[:op.n_fe] for B in (u + v, u, v))
    assert (Yu.abs() > 0).all() and Yv.abs().max() > 0
    assert torch.equal(Y, Yu + Yv)
