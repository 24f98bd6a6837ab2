"""The fold of the tile partials inside the enrichment chain (at most 64 partials of a function), eight list
entries at a time: lists of 4, 8, 16, 27, 43 and 64 tiles, in the chain's own launch and as part of the cell
launch, against the oracle.

Tolerances as for the other comparisons with the oracle: 1e-10 per column in float64, 5e-5 in float32."""
import numpy as np
import pytest

from oracle import chfsi as och
from oracle.operator import OEFEOperator
from paper_2010_09701_amd import workloads as wl

pytestmark = pytest.mark.gpu

K = np.array([0.21, -0.37, 0.13])


def _colrel(A, B):
    return float((np.linalg.norm(A - B, axis=0) / np.linalg.norm(B, axis=0)).max())


@pytest.mark.parametrize("nc", [3, 4, 5, 6, 7, 8])  # (2 nc)^3 / 64 tiles of 64 rows
@pytest.mark.parametrize("cplx", [False, True])
def test_folded_partials(nc, cplx):
    import torch
    from paper_2010_09701_amd import oefe
    sysm = wl.tiny_system(nc=nc, p=2, n_atoms=3, seed=17, L=6.0, r0=1.2, r1=2.9)
    if cplx:
        sysm = sysm.with_k(K)
    op, gop = OEFEOperator(sysm), oefe.Operator(sysm)
    X = wl.start_block(op.n_tot, 19, 5, complex_=cplx)
    a0, b, _, _ = och.lanczos_bounds(op.apply, wl.lanczos_start(op.n_tot, 2), 10)
    a = 0.5 * (a0 + b)
    Y, F = op.apply(X), och.chebyshev_filter(op.apply, X, 3, a, b, a0)
    for single in (False, True):
        dt, tol = (("complex64" if cplx else "float32"), 5e-5) if single else (("complex128" if cplx else "float64"), 1e-10)
        for nv in (1, 2, 19):
            Xd = torch.from_numpy(np.ascontiguousarray(X[:, :nv])).to(getattr(torch, dt)).cuda()
            assert _colrel(oefe.ham_apply(gop, Xd).cpu().numpy(), Y[:, :nv]) < tol, (dt, nv)
            assert _colrel(oefe.chebyshev_filter(gop, Xd, 3, a, b, a0).cpu().numpy(), F[:, :nv]) < tol, (dt, nv)
