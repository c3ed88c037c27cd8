"""Relaxation parameters of a node list from its runs along x, where the division
into runs can go wrong: gaps in a row, rows with two cell sizes, a row of one node,
the same node twice, more than 64 x coordinates (two table chunks), nodes in no
order, two shapes (nitrogen); and a list that falls into no runs.  One pass from a
seeded random VDF against the FP64 oracle.

Tolerance: that of the list's one-pass parity test, 1e-13 of the largest value.  A
run's sum is a difference of prefix sums of at most 90 terms, 90 x 1.1e-16 of the
whole row's at worst and 1e-15 in the sum over rows, where the errors are of either
sign; the 5 x 5 system for the conservation terms (condition number below 50)
keeps that below 5e-14.
"""
import dataclasses

import numpy as np
import pytest

from oracle.oracle import Oracle
from paper_2310_18916_amd import inputs as I

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2310_18916_amd.gsis import Solver  # noqa: E402


def lattice(n, vmax=4.0):
    return I.tensor_velocity_list(n, (-vmax,) * 3, (vmax,) * 3)


def gaps():
    a = lattice((19, 9, 8))
    keep = np.random.default_rng(1).random(a.shape[0]) > 0.1
    keep[19 * 3:19 * 4] = False
    keep[19 * 3 + 5] = True    # a row of one node
    return a[keep]


def twice():
    a = lattice((17, 8, 7))
    b = a[100:140].copy()
    a[100:140, 3] *= 0.5       # two halves of a node count once
    b[:, 3] *= 0.5
    return np.concatenate([a, b])


def shuffled(a, seed=3):
    return np.ascontiguousarray(a[np.random.default_rng(seed).permutation(a.shape[0])])


def scattered():
    a = lattice((12, 9, 8))
    a[:, :3] += np.random.default_rng(2).uniform(-0.1, 0.1, (a.shape[0], 3))
    return a


LISTS = {
    "gaps": gaps(),
    "twice": twice(),
    "two_sizes": shuffled(I.hypersonic_velocity_mesh(2.0, 5.0 / 3.0, 1.0)),
    "long_rows": shuffled(lattice((90, 8, 7))),
    "table_edge": lattice((64, 6, 7)),
    "no_runs": scattered(),
}


@pytest.mark.parametrize("species", [I.MONATOMIC, I.DIATOMIC])
@pytest.mark.parametrize("name", list(LISTS))
def test_runs(name, species):
    case = I.small_block(species=species, n=(6, 5, 4), blk=((2, 4), (2, 3), (1, 3)))
    case = I.with_velocity_list(dataclasses.replace(case, conservative=1), LISTS[name])
    print(name, species, case.nvel, flush=True)
    f0, f1 = I.random_vdf(case, seed=9)
    o = Oracle(case)
    o.set_vdf(f0, f1)
    assert o.step(1) == 0
    s = Solver(case, "fp64")
    s.set_vdf(f0, f1)
    s.kinetic_step(1)
    fluid = ~case.solid_mask().astype(bool)
    for a, b in zip(s.get_vdf(), o.get_vdf()):
        if b is not None:
            a, b = a.cpu().numpy()[fluid], b[fluid]
            assert np.abs(a - b).max() / np.abs(b).max() <= 1e-13
