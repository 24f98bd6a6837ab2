"""First step of a float32 recurrence (the tile partials of its start block, formed by a kernel of their own)
on meshes whose last tiles hold at most 32 rows, so that one wave of a column group has no row at all:
the same bits with 1, 2 and 4 column groups to a workgroup, and the oracle's filter.

Tolerance as for the other float32 comparisons with the oracle: 5e-5 per column."""
import numpy as np
import pytest

from oracle import chfsi as och
from oracle.operator import OEFEOperator
from paper_2010_09701_amd import workloads as wl

pytestmark = pytest.mark.gpu

K = np.array([0.21, -0.37, 0.13])


@pytest.mark.parametrize("nc,p", [(3, 2), (3, 3)])  # 6^3 = 3 * 64 + 24 rows, 9^3 = 11 * 64 + 25 rows
@pytest.mark.parametrize("dt,nv", [("float32", 32), ("float32", 96), ("complex64", 16), ("complex64", 41)])
def test_first_step_partials_ragged_tiles(nc, p, dt, nv):
    import torch
    from paper_2010_09701_amd import oefe
    cplx = dt == "complex64"
    sysm = wl.tiny_system(nc=nc, p=p, n_atoms=2, seed=11, L=7.0, r0=1.0, r1=2.5)
    if cplx:
        sysm = sysm.with_k(K)
    op, gop = OEFEOperator(sysm), oefe.Operator(sysm)
    X = wl.start_block(op.n_tot, nv, 5, complex_=cplx).astype(np.complex64 if cplx else np.float32)
    a0, b, _, _ = och.lanczos_bounds(op.apply, wl.lanczos_start(op.n_tot, 2), 10)
    a = 0.5 * (a0 + b)
    ref = och.chebyshev_filter(op.apply, X.astype(np.complex128 if cplx else np.float64), 3, a, b, a0)
    Xd = torch.from_numpy(X).cuda()
    Y = oefe.chebyshev_filter(gop, Xd.clone(), 3, a, b, a0)
    err = np.linalg.norm(Y.cpu().numpy() - ref, axis=0) / np.linalg.norm(ref, axis=0)
    assert err.max() < 5e-5, err.max()
    for cb in (16, 32, 64):
        oefe.set_launch_shape(gop, 0, cb)
        assert torch.equal(oefe.chebyshev_filter(gop, Xd.clone(), 3, a, b, a0), Y), cb
