"""The moment sums of the stored VDF where their loads and table can go wrong: octants
shorter than a load, a chunk and a stretch of a row, and one node over each; octants of
very different sizes and one without a node; cells one over a wave's 16 and a block's
64; solid cells; two VDFs; a node list.

Against extended precision on the CPU: a sum is at most 20 roundings in a chunk and
segment and a compensated addition per segment, of terms with two or three roundings
each, 2.5e-15 of the sum of their magnitudes; 1e-14 leaves a factor 4.
"""
import dataclasses

import numpy as np
import pytest

from oracle.oracle import node_grid
from paper_2310_18916_amd import inputs as I

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2310_18916_amd.gsis import Solver  # noqa: E402

GAS = {"species": I.DIATOMIC, "dr": I.N2_DR, "Zr": I.N2_ZR, "A": I.N2_A}


def box(n, m, **kw):
    c = dataclasses.replace(I.cavity(4, 4, 0.1, lid=0.2), **kw)
    c.nx, c.ny, c.nz, c.nv = *n, m
    return c


def octants(sizes, seed=5):
    """A node list with the given number of nodes per octant."""
    rng = np.random.default_rng(seed)
    out = []
    for o, k in enumerate(sizes):
        x = rng.uniform(0.05, 3.5, (k, 3)) * [-1.0 if (o >> a) & 1 else 1.0 for a in range(3)]
        out.append(np.column_stack([x, rng.uniform(0.5, 2.0, k)]))
    return np.concatenate(out)


CASES = {
    "one_node": box((3, 3, 2), (2, 2, 2)),
    "odd": box((17, 2, 2), (5, 7, 9)),
    "chunk": box((13, 5, 1), (8, 8, 8)),
    "stretch": box((5, 4, 4), (8, 8, 16)),
    "over": box((9, 9, 1), (9, 9, 9)),
    "two_vdfs": box((5, 5, 3), (11, 8, 10), **GAS),
    "edges": I.with_velocity_list(box((13, 5, 1), (2, 2, 2)), octants([1, 3, 63, 64, 65, 127, 129, 257])),
    "empty": I.with_velocity_list(box((4, 4, 1), (2, 2, 2)), octants([0, 2, 128, 130, 256, 5, 191, 300])),
    "solid": I.small_block(species=I.DIATOMIC, n=(6, 5, 4), blk=((2, 4), (2, 3), (1, 3))),
}


@pytest.mark.parametrize("dtype", ["fp64", "fp32"])
@pytest.mark.parametrize("name", list(CASES))
def test_moments(name, dtype):
    case = CASES[name]
    print(name, dtype, case.ncell, case.nvel, flush=True)
    rng = np.random.default_rng(11)
    f0 = rng.uniform(0.1, 1.0, (case.ncell, case.nvel))
    f1 = rng.uniform(0.1, 1.0, f0.shape) if case.species == I.DIATOMIC else None
    if dtype == "fp32":
        f0 = f0.astype(np.float32).astype(np.float64)
        f1 = f1 if f1 is None else f1.astype(np.float32).astype(np.float64)
    live = np.ones(case.ncell, bool) if case.solid is None else np.asarray(case.solid).reshape(-1) == 0
    s = Solver(case, dtype)
    s.set_vdf(f0, f1)
    got = s.moments()[live]
    xi, w = (np.asarray(a, np.longdouble) for a in node_grid(case))
    f0, c2 = f0[live].astype(np.longdouble), (xi * xi).sum(1)
    rho = f0 @ w
    mean = lambda m: (f0 @ (w * m)) / rho               # noqa: E731
    size = lambda m: (f0 @ (w * np.abs(m))) / rho       # noqa: E731
    near = lambda a, b, scale: np.abs(a - b).max() <= 1e-14 * scale.max()     # noqa: E731
    assert near(got[:, 0], rho, rho)
    u = np.stack([mean(xi[:, a]) for a in range(3)], 1)
    for a in range(3):
        assert near(got[:, 1 + a], u[:, a], size(xi[:, a]))
    e = mean(c2)
    assert near(got[:, 4], (e - (u * u).sum(1)) * 2 / 3, e)
    q = np.stack([mean(xi[:, a] * c2) - 2 * sum(mean(xi[:, a] * xi[:, b]) * u[:, b] for b in range(3)) - u[:, a] * e
                  + 2 * u[:, a] * (u * u).sum(1) for a in range(3)], 1) * rho[:, None]
    for a in range(3):
        assert near(got[:, 11 + a], q[:, a], 8 * rho * size(np.abs(xi).max(1) * c2))
    if case.species == I.DIATOMIC:
        f1 = f1[live].astype(np.longdouble)
        e1 = f1 @ w
        assert near(got[:, 14], 2 * e1 / (case.dr * rho), e1 / rho)
        for a in range(3):
            assert near(got[:, 15 + a], f1 @ (w * xi[:, a]) - u[:, a] * e1, 4 * (f1 @ (w * np.abs(xi).max(1))))
