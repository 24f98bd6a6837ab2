"""What the host code queues and refuses, on the CPU with a recording HIP runtime."""
import dataclasses

import numpy as np
import pytest

from paper_2010_09701_amd import workloads as wl

F64, C128 = 0, 3
EINVAL = -1


@pytest.fixture(scope="module")
def rec(tmp_path_factory):
    from recorded import Recorded
    return Recorded(str(tmp_path_factory.mktemp("recorded")))


def test_batch_of_unlike_operators_is_refused(rec):
    """A Kohn-Sham operator with one function per atom and the auxiliary-potential operator of the same atoms
    have the same mesh and coupling lists, but store their coupling blocks with different row strides: one
    launch cannot serve both."""
    base = wl.tiny_system(nc=3, p=2, n_atoms=3, seed=13, L=6.0, r0=1.0, r1=2.3)
    s = dataclasses.replace(base, enr=[wl.EnrichmentFn(a, 0, 2.0, -1) for a in range(3)])
    ks, pois = rec.operator(s), rec.operator(s, poisson=True)
    n_tot = s.n_fe + 3
    assert rec.batched([ks, ks], F64, n_tot, 4, 2) == 0 and rec.batched([pois, pois], F64, n_tot, 4, 2) == 0
    rec.events()
    for pair in ([ks, pois], [pois, ks]):
        assert rec.batched(pair, F64, n_tot, 4, 2) == EINVAL
        assert rec.autotune(pair, F64, n_tot, 4)[0] == EINVAL
        assert rec.events() == []


@pytest.mark.parametrize("m", [1, 3])
def test_failed_node_launch_leaves_no_side_work(rec, m):
    """A step whose node kernel cannot be launched returns with its enrichment chain queued on the side
    stream: the caller's stream has to wait for it, because the chain writes into the caller's buffers."""
    base = wl.tiny_system(nc=3, p=2, n_atoms=8, seed=13, L=6.0, r0=1.0, r1=2.9)
    enr = [wl.EnrichmentFn(a, i // 4, 2.0 / (1 + i % 4), (i % 4) - 1) for a in range(8) for i in range(8)]
    s = dataclasses.replace(base, enr=enr).with_k(np.array([0.21, -0.37, 0.13]))
    op = rec.operator(s)  # 64 complex functions: chain and fold on the side stream, more than 64 KB of LDS a tile
    rec.events()
    rec.fail_attribute("fe_node_kernel")
    try:
        assert rec.filter(op, C128, s.n_tot, 1, m, stream=7) != 0
    finally:
        rec.fail_attribute()
    ev = rec.events()
    side = [i for i, e in enumerate(ev) if type(e).__name__ == "Launch" and e.stream != 7]
    assert side and not any(type(e).__name__ == "Launch" and "fe_node_kernel" in e.kernel for e in ev)
    joined = [i for i, e in enumerate(ev) if type(e).__name__ == "Record" and e.stream == ev[side[-1]].stream and i > side[-1]]
    assert joined and any(type(e).__name__ == "Wait" and e.stream == 7 and e.event == ev[joined[-1]].event
                          for e in ev[joined[-1]:])


def _launches(ev, name):
    return [e for e in ev if type(e).__name__ == "Launch" and name in e.kernel]


@pytest.mark.parametrize("nc,p,nv,nfn,in_cell", [(8, 2, 16, 5, True), (12, 2, 64, 5, False), (12, 2, 64, 3, True),
                                                 (7, 4, 37, 5, True)])
def test_chain_in_cell_launch_of_a_bloch_operator(rec, nc, p, nv, nfn, in_cell):
    """Where a complex128 step's enrichment chain runs.  As the first blocks of the cell launch it holds that
    launch's LDS and registers, which 40 functions (59 KB, two workgroups a CU) may do for a small step only:
    a step of 1.8 M elements of degree 2 takes the side stream, and its cell kernel is the instance without the chain."""
    enr = [wl.EnrichmentFn(a, i // 4, 14.0 / (1 + i % 4), (i % 4) - 1) for a in range(8) for i in range(nfn)]
    s = dataclasses.replace(wl.diamond8(nc=nc, p=p), enr=enr).with_k(np.array([0.21, -0.37, 0.13]))
    op = rec.operator(s)
    rec.events()
    assert rec.filter(op, C128, s.n_tot, nv, 4) == 0
    ev = rec.events()
    cells = _launches(ev, "fe_cell_lanes_kernel")
    assert len(cells) == 4 and all(c.stream == 7 for c in cells)
    assert bool([e for e in ev if type(e).__name__ == "Launch" and e.stream != 7]) == (not in_cell)
    for c in cells:
        # workgroups of 256 threads by LDS: the cell tile's 21 KB (static, 0 here) or the chain's
        assert (c.lds == 0) == (not in_cell)
    assert len({c.kernel for c in cells}) == 1


@pytest.mark.parametrize("nc,nv,groups", [(6, 16, 1), (12, 8, 1), (12, 72, 2), (12, 320, 4)])
def test_node_workgroups_of_small_launches(rec, nc, nv, groups):
    """Column groups of a node workgroup (two waves each) by the size of the launch: 27 tiles of one group and 216
    of one would leave most CUs idle with workgroups of four, 216 tiles of five groups with workgroups of four."""
    s = wl.diamond8(nc=nc, p=2)
    op = rec.operator(s)
    rec.events()
    assert rec.filter(op, F64, s.n_tot, nv, 2) == 0
    nodes = _launches(rec.events(), "fe_node_kernel")
    assert [e.block for e in nodes] == [128 * groups] * 2


@pytest.mark.parametrize("atoms,one_workgroup", [(250, True), (260, False)])
def test_one_column_of_many_functions(rec, atoms, one_workgroup):
    """One workgroup forms the enrichment rows of a column up to 256 functions; beyond, reading both matrices alone
    takes it longer than the launches of many workgroups."""
    g = (np.arange(7) + 0.5) * 3.0
    pos = np.stack(np.meshgrid(g, g, g, indexing="ij"), -1).reshape(-1, 3)[:atoms]
    s = wl.System("lattice", 21.0, 10, 2, pos, np.full(atoms, 3.0), 0.5, 0.8, 1.4, [])
    op = rec.operator(s, poisson=True)
    rec.events()
    assert rec.apply(op, F64, s.n_fe + atoms, 1) == 0
    ev = rec.events()
    assert bool(_launches(ev, "enr_col1_kernel")) == one_workgroup
    assert bool(_launches(ev, "small_gemm_kernel")) == (not one_workgroup)


@pytest.mark.parametrize("nc", [3, 12])
def test_autotuner_times_the_steps_of_a_filter(rec, nc):
    """The launch-shape tuner times steps like those in the middle of a filter, whose node kernel forms the next
    step's partials: between its timing events no start-up work of a recurrence (partials of the given block,
    Z^O) is queued, and a shape is timed once."""
    s = wl.diamond8(nc=nc, p=2) if nc > 3 else wl.tiny_system(nc=nc, p=2, n_atoms=2, seed=13, L=6.0, r0=1.0, r1=2.3)
    op = rec.operator(s)
    rec.events()
    rc, cw, cb = rec.autotune([op], F64, s.n_tot, 40, reps=5)
    assert rc == 0 and cw in (0, 8, 16, 32, 64) and cb in (16, 32, 64)
    ev = rec.events()
    # the events recorded on the stream that no stream waits for are the timing events, in pairs
    waited = {e.event for e in ev if type(e).__name__ == "Wait"}
    marks = [i for i, e in enumerate(ev) if type(e).__name__ == "Record" and e.stream == 7 and e.event not in waited]
    assert len(marks) == 2 * 5 * 3
    shapes = set()
    for a, b in zip(marks[::2], marks[1::2]):
        nodes, cells = _launches(ev[a:b], "fe_node_kernel"), _launches(ev[a:b], "fe_cell")
        assert len(nodes) == 5 and not _launches(ev[a:b], "fe_part_kernel")
        assert all("ELi1ELb0EEEv" in n.kernel for n in nodes)  # partials from the result, not from the step's X
        shapes.add((cells[0].kernel, cells[0].grid, nodes[0].block))
    assert len(shapes) == 15
