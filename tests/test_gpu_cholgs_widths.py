"""CholGS at the widths where its kernels change: complex blocks below and above 8 columns (Gram matrix
as the real one of the interleaved columns), around 40 (in-place product), and at the last sizes of each
factorization (complex 70 and 128, real 100 and 160 columns, and the steps of 32 columns between).

The factor R of X = Q R with a positive diagonal is unique, so Q is compared with LAPACK's QR, its
phases removed.  Random blocks with uniform entries have condition numbers below 10 at these shapes
(n >= 3 nv), and CholGS errs by a small multiple of eps cond^2 nv < 2.2e-16 * 100 * 161 = 4e-12."""
import numpy as np
import pytest

from paper_2010_09701_amd import workloads as wl

pytestmark = pytest.mark.gpu

K = np.array([0.21, -0.37, 0.13])


@pytest.mark.parametrize("nc", [4, 8])  # 512 rows, and enough rows for the wide products (4096)
@pytest.mark.parametrize("nv", [1, 7, 8, 9, 40, 41, 70, 71, 96, 97, 128, 129])
@pytest.mark.parametrize("cplx", [True, False])
def test_cholgs_widths(nc, nv, cplx):
    import torch
    from paper_2010_09701_amd import oefe
    if not cplx:
        nv += 32 if nv > 70 else 30 if nv == 70 else 0  # 100, 103, 128, 129, 160, 161
    sysm = wl.tiny_system(nc=nc, p=2, n_atoms=2, seed=13, L=6.0, r0=1.0, r1=2.3)
    op = oefe.Operator(sysm.with_k(K) if cplx else sysm)
    X = wl.start_block(op.n_tot, nv, 3, complex_=cplx)
    Q, R = np.linalg.qr(X)
    Q = Q * (np.diag(R) / np.abs(np.diag(R)))
    Xd = torch.from_numpy(X).cuda()
    oefe.cholgs(op, Xd)
    err = np.abs(Xd.cpu().numpy() - Q).max()
    assert err < 4e-12, err
    # a column that repeats an earlier one breaks down there, whichever kernel factors
    if nv > 7:
        X[:, nv - 2] = X[:, 1]
        with pytest.raises(RuntimeError, match=f"column {nv - 2}"):
            oefe.cholgs(op, torch.from_numpy(X).cuda())


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
