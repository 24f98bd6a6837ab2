"""The node stage at the edges of its column groups (16 real columns in float64, 32 in float32, up to four
groups a workgroup, workgroups across tile ends) and of its tiles: one application (partials of X) and a
two-step filter (partials of the step's result, two Z^O buffers) against the oracle, for block widths
around 16, 32 and 64 real columns (one column: kernels of its own), on meshes with ragged tiles, x-lines that do not end with a tile's
rows, and Bloch phases.

Tolerances as for the other comparisons with the oracle: 1e-10 per column in float64, 5e-5 in float32
(float32 rounding times the spread of the operator)."""
import numpy as np
import pytest

from oracle import chfsi as och
from oracle.operator import OEFEOperator
from paper_2010_09701_amd import workloads as wl

pytestmark = pytest.mark.gpu

K = np.array([0.21, -0.37, 0.13])
SYSTEMS = {
    "atom": lambda: wl.single_atom(),                                                          # n = 8
    "p3": lambda: wl.tiny_system(nc=3, p=3, n_atoms=2, seed=11, L=7.0, r0=1.0, r1=2.5),        # n = 9
    "diamond_nc5": lambda: wl.diamond8(nc=5, p=4),                                             # n = 20
    "free": lambda: wl.free_system(6.0, 3, 3),                                                 # no enrichment
}
WIDTHS = {"real": (1, 2, 15, 16, 17, 31, 33, 63, 64, 65, 81), "cplx": (1, 7, 8, 9, 16, 17, 31, 33, 41)}


def _colrel(A, B):
    return float((np.linalg.norm(A - B, axis=0) / np.maximum(np.linalg.norm(B, axis=0), 1e-300)).max())


@pytest.mark.parametrize("name", sorted(SYSTEMS))
@pytest.mark.parametrize("dt", ["float64", "float32", "complex128", "complex64"])
def test_node_stage_column_groups(name, dt):
    import torch
    from paper_2010_09701_amd import oefe
    cplx = dt.startswith("complex")
    single = dt in ("float32", "complex64")
    sysm = SYSTEMS[name]() if not cplx else SYSTEMS[name]().with_k(K)
    op, gop = OEFEOperator(sysm), oefe.Operator(sysm)
    widths = WIDTHS["cplx" if cplx else "real"]
    X = wl.start_block(op.n_tot, max(widths), 5, complex_=cplx)
    if single:
        X = X.astype(np.complex64 if cplx else np.float32).astype(X.dtype)
    a0, b, _, _ = och.lanczos_bounds(op.apply, wl.lanczos_start(op.n_tot, 2), 10)
    a = 0.5 * (a0 + b)
    Y, F = op.apply(X), och.chebyshev_filter(op.apply, X, 2, a, b, a0)
    tol = 5e-5 if single else 1e-10
    for nv in widths:
        Xd = torch.from_numpy(np.ascontiguousarray(X[:, :nv])).to(getattr(torch, dt)).cuda()
        assert _colrel(oefe.ham_apply(gop, Xd).cpu().numpy(), Y[:, :nv]) < tol, nv
        oefe.chebyshev_filter(gop, Xd, 2, a, b, a0)
        assert _colrel(Xd.cpu().numpy(), F[:, :nv]) < tol, nv


@pytest.mark.parametrize("dt,nv,sub", [("float64", 181, (2, 3, 4, 5, 64)), ("float32", 181, (2, 33)),
                                       ("complex128", 92, (2, 5, 17)), ("complex64", 92, (2, 33))])
def test_recurrence_enrichment_chain_placement(dt, nv, sub):
    """A recurrence whose blocks hold more than 2^23 real elements runs the enrichment chain on the side
    stream, a smaller one in the cell launch: the same sums in the same order, so the columns of a wide
    block and of narrow ones are equal to the bit."""
    import torch
    from paper_2010_09701_amd import oefe
    sysm = wl.diamond8(nc=9, p=4)
    op = oefe.Operator(sysm.with_k(K) if dt.startswith("complex") else sysm)
    assert op.n_tot * nv * (2 if dt.startswith("complex") else 1) > 1 << 23
    X = torch.from_numpy(wl.start_block(op.n_tot, nv, 5, complex_=dt.startswith("complex"))).to(getattr(torch, dt)).cuda()
    a0, b = oefe.lanczos_bounds(op, torch.from_numpy(wl.lanczos_start(op.n_tot, 2)).cuda(), 10)[:2]
    wide = oefe.chebyshev_filter(op, X.clone(), 5, 0.5 * (a0 + b), b, a0)
    for w in sub:
        narrow = oefe.chebyshev_filter(op, X[:, :w].contiguous(), 5, 0.5 * (a0 + b), b, a0)
        assert torch.equal(narrow, wide[:, :w]), w
