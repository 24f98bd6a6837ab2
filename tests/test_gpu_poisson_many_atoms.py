"""The auxiliary potential of more than 256 atoms: the enrichment products of a conjugate-gradient step in launches
of many workgroups, and p . q by a pass of its own; 250 atoms on the same mesh take the single workgroup.

Tolerances as for the other comparisons with the oracle: the operator 1e-10, the solution 1e-8 of its largest
coefficient (the steps stop at a relative residual of 1e-12, condition numbers below 1e4)."""
import numpy as np
import pytest

from oracle import poisson as po
from paper_2010_09701_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("atoms", [250, 260])
def test_many_atoms(atoms):
    import torch
    from paper_2010_09701_amd import oefe
    k, a = 7, 3.0
    g = (np.arange(k) + 0.5) * a
    pos = np.stack(np.meshgrid(g, g, g, indexing="ij"), -1).reshape(-1, 3)
    pos += np.random.default_rng(1).uniform(-0.2, 0.2, pos.shape)
    s = wl.System("lattice", k * a, 10, 2, pos[:atoms] % (k * a), np.full(atoms, 3.0), 0.5, 0.8, 1.4, [])
    P, pop = po.PoissonOEFE(s), oefe.Operator(s, poisson=True)
    lam, U = np.linalg.eigh(P.Aoo)
    S, d = (U / np.sqrt(lam)[None, :]) @ U.T, 1.0 / np.sqrt(P.m)
    X = np.random.default_rng(3).uniform(-1.0, 1.0, size=(P.n_tot, 3))
    AZ = P.matrix() @ np.concatenate([d[:, None] * X[:P.N], S @ X[P.N:]])
    Yo = np.concatenate([d[:, None] * AZ[:P.N], S @ AZ[P.N:]])
    for c in (1, 3):
        Y = oefe.ham_apply(pop, torch.from_numpy(np.ascontiguousarray(X[:, :c])).cuda()).cpu().numpy()
        assert (np.abs(Y - Yo[:, :c]).max(axis=0) / np.abs(Yo[:, :c]).max(axis=0)).max() <= 1e-10, c
    rho = P.model_electron_density()
    phi_o = P.solve(P.neutral_charge(rho))
    phi, it, rel = oefe.poisson_solve(pop, torch.from_numpy(np.ascontiguousarray(rho)).cuda(), tol=1e-12, max_iter=5000)
    assert rel <= 1e-12 and 0 < it < 5000
    assert np.abs(phi.cpu().numpy() - phi_o).max() <= 1e-8 * np.abs(phi_o).max()
