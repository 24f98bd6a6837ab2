"""What the host code queues and refuses, on the CPU with a recording HIP runtime."""
import dataclasses

import numpy as np
import pytest

from paper_2010_09701_amd import workloads as wl

F64, C128 = 0, 3
EINVAL = -1


@pytest.fixture(scope="module")
def rec():
    from recorded import Recorded
    return Recorded()


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
