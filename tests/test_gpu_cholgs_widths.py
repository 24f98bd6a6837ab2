"""CholGS of blocks wider than the one-workgroup factorizations.

The factor R of X = Q R with a positive diagonal is unique, so Q is compared with LAPACK's QR, its
phases removed.  Random blocks with uniform entries have condition numbers below 10 at these shapes
(n >= 3 nv), and CholGS errs by a small multiple of eps cond^2 nv < 2.2e-16 * 100 * 170 = 4e-12."""
import numpy as np
import pytest

from paper_2010_09701_amd import workloads as wl

pytestmark = pytest.mark.gpu

K = np.array([0.21, -0.37, 0.13])


@pytest.mark.parametrize("cplx", [True, False])
def test_cholgs_wide_repeats(cplx):
    """Above the one-workgroup sizes: the same block gives the same bits every time (the scaling of the
    Gram matrix by its diagonal must not read a diagonal entry that is already scaled)."""
    import torch
    from paper_2010_09701_amd import oefe
    sysm = wl.tiny_system(nc=4, p=2, n_atoms=2, seed=13, L=6.0, r0=1.0, r1=2.3)
    op = oefe.Operator(sysm.with_k(K) if cplx else sysm)
    X = wl.start_block(op.n_tot, 170, 3, complex_=cplx)
    Q, R = np.linalg.qr(X)
    Q = Q * (np.diag(R) / np.abs(np.diag(R)))
    X = torch.from_numpy(X).cuda()
    ref = oefe.cholgs(op, X.clone())
    assert np.abs(ref.cpu().numpy() - Q).max() < 4e-12
    for _ in range(20):
        assert torch.equal(oefe.cholgs(op, X.clone()), ref)
