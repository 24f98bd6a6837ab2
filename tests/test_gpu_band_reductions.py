"""The reductions of the band energy at the widths where their split changes: sum_j f_j Re(x_j . y_j) for
block widths around 64, 128 and 256 columns (whole rows to a workgroup, a second group of columns above
256) with padded rows, float64 / float32 / complex blocks.

Float64 sums of n nv < 2e5 terms of size below 1 in any order agree to n nv eps sum|terms| / n nv < 1e-11
of the sum of their sizes; products of float32 entries are exact in float64."""
import numpy as np
import pytest

from paper_2010_09701_amd import workloads as wl

pytestmark = pytest.mark.gpu

K = np.array([0.21, -0.37, 0.13])


@pytest.mark.parametrize("dt", ["float64", "float32", "complex128", "complex64"])
def test_band_energy_widths(dt):
    import torch
    from paper_2010_09701_amd import oefe
    cplx, single = dt.startswith("complex"), dt in ("float32", "complex64")
    sysm = wl.single_atom() if not cplx else wl.single_atom().with_k(K)
    op = oefe.Operator(sysm)
    for nv in (1, 2, 63, 65, 127, 129, 255, 256, 257):
        X = wl.start_block(op.n_tot, nv, 4, complex_=cplx).astype(dt)
        f = wl.occupations(nv, 3)
        Xd = torch.zeros(op.n_tot, nv + 3, dtype=getattr(torch, dt), device="cuda")[:, :nv]
        Xd.copy_(torch.from_numpy(X))
        HX = oefe.ham_apply(op, Xd.contiguous()).cpu().numpy().astype(np.complex128 if cplx else np.float64)
        terms = np.real(np.conj(X.astype(HX.dtype)) * HX) * f
        E = oefe.band_energy_grad(op, Xd, torch.from_numpy(f).cuda())[0]
        assert abs(float(E) - terms.sum()) < 1e-11 * np.abs(terms).sum(), nv


def test_band_energy_gradient_padded_rows():
    """dE/dX of a block with padded rows has the block's row stride (the library writes with it)."""
    import torch
    from paper_2010_09701_amd import oefe
    op = oefe.Operator(wl.single_atom())
    X = torch.from_numpy(wl.start_block(op.n_tot, 5, 4)).cuda()
    f = torch.from_numpy(wl.occupations(5, 3)).cuda()
    Xp = torch.zeros(op.n_tot, 8, dtype=X.dtype, device="cuda")[:, :5]
    Xp.copy_(X)
    _, _, dX = oefe.band_energy_grad(op, X, f)
    _, _, dXp = oefe.band_energy_grad(op, Xp, f)
    assert dXp.stride() == (8, 1) and torch.equal(dX, dXp)


@pytest.mark.parametrize("kvec", [None, (0.21, -0.37, 0.13)])
@pytest.mark.parametrize("nfn", [(1, 1), (3, 1), (4, 4), (6, 2), (7, 5), (8, 8)])
def test_functions_per_atom(nfn, kvec):
    """The potential rebuild (H^oo of block pairs with 1..8 functions, equal and unequal) and, for it and
    the gradient in the potential, the enrichment part at the points: against the oracle as in the
    other comparisons (1e-10 per column; the gradient 1e-10 relative, 1e-12 of its largest entry)."""
    import dataclasses

    import torch
    from oracle import adjoint as adj
    from oracle.operator import OEFEOperator
    from paper_2010_09701_amd import oefe
    base = wl.tiny_system(nc=3, p=2, n_atoms=2, seed=13, L=6.0, r0=1.0, r1=2.3)
    fns = [wl.EnrichmentFn(a, i // 4, 2.0 / (1 + i % 4), (i % 4) - 1) for a in (0, 1) for i in range(nfn[a])]
    sysm = dataclasses.replace(base, enr=fns)
    if kvec is not None:
        sysm = sysm.with_k(np.array(kvec))
    op0, gop = OEFEOperator(sysm), oefe.Operator(sysm)
    V = op0.V + 0.3 * wl.potential_perturbation(op0.mesh.n_cells, op0.mesh.nq, 101)
    gop.set_potential(torch.from_numpy(V).cuda())
    op = OEFEOperator(sysm, V=V)
    X = wl.start_block(op.n_tot, 19, 2, complex_=kvec is not None)
    Xd = torch.from_numpy(X).cuda()
    Y, ref = oefe.ham_apply(gop, Xd).cpu().numpy(), op.apply(X)
    assert (np.linalg.norm(Y - ref, axis=0) / np.linalg.norm(ref, axis=0)).max() < 1e-10
    f = wl.occupations(19, 3)
    dV = oefe.band_energy_grad(gop, Xd, torch.from_numpy(f))[1].cpu().numpy()
    gv = adj.grad_V(op, X, f)
    np.testing.assert_allclose(dV, gv, rtol=1e-10, atol=1e-12 * np.abs(gv).max())
