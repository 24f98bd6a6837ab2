"""dE/dX of a block with padded rows."""
import pytest

from paper_2010_09701_amd import workloads as wl

pytestmark = pytest.mark.gpu


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
