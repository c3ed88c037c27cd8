"""Moment sums formed in the sweep (states over 256 MB), at the sizes where their
chunks and segments can go wrong: octants that end inside a chunk, in a segment's
first and last chunk; boxes one cell over a tile and thinner than one; solid cells;
two VDFs; a per-point term; a node list; two precisions; a batch.

Against the sums from the stored VDF (the 4 x 4 x 4 tile with 128 threads, whose
sweep forms none): the same chunks in the same order, so bitwise.  Against a plain
FP64 product of the stored VDF with the nodes: a sum is 16 + 4 roundings in a chunk
and segment and one per segment, at most 450 here, each 1.1e-16 of a sum of
positive terms (density, energy), 5e-14; 1e-12 leaves a factor 20.
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

from paper_2310_18916_amd.gsis import Batch, Solver  # noqa: E402


def box(n, m, **kw):
    c = dataclasses.replace(I.cavity(4, 4, 0.1, lid=0.2), **kw)
    c.nx, c.ny, c.nz, c.nv = *n, m
    return c


def solid(species):
    c = I.block_flow(9, 8, 7, ((3, 6), (2, 6), (3, 5)), 10, 5.0, 0.3, Ma=0.5, species=species)
    c.nv = (42, 41, 40)
    return c


def refined():
    c = I.block_flow(17, 16, 17, ((6, 10), (6, 10), (6, 9)), 4, 12.0, 0.1, Ma=5.0)
    return I.with_velocity_list(c, I.hypersonic_velocity_mesh(5.0, 5.0 / 3.0, 1.0))


GAS = {"species": I.DIATOMIC, "dr": I.N2_DR, "Zr": I.N2_ZR, "A": I.N2_A}
CASES = {
    "whole": (lambda: box((4, 4, 4), (88, 96, 96)), "fp64"),
    "over": (lambda: box((5, 4, 3), (90, 89, 91)), "fp64"),
    "over_fp32": (lambda: box((5, 9, 3), (90, 89, 91)), "fp32"),
    "over_fp32_8x4": (lambda: box((11, 5, 9), (60, 61, 59)), "fp32"),
    "thin": (lambda: box((1, 1, 29), (118, 97, 102)), "fp64"),
    "few_nodes": (lambda: box((83, 81, 82), (4, 4, 4)), "fp64"),
    "term": (lambda: box((5, 4, 3), (90, 89, 91), inv_dt=3.0), "fp64"),
    "second_order": (lambda: box((6, 5, 4), (70, 71, 69), order=2), "fp64"),
    "solid": (lambda: solid(I.MONATOMIC), "fp64"),
    "solid_fp32": (lambda: dataclasses.replace(solid(I.MONATOMIC), nv=(52, 51, 53)), "fp32"),
    "two_vdfs": (lambda: box((5, 5, 3), (70, 71, 69), **GAS), "fp64"),
    "two_vdfs_solid": (lambda: solid(I.DIATOMIC), "fp64"),
    "two_vdfs_wide": (lambda: box((16, 12, 12), (44, 44, 42), **GAS), "fp64"),
    "two_vdfs_fp32": (lambda: box((5, 5, 5), (70, 71, 69), **GAS), "fp32"),
    "list": (refined, "fp64"),
    "list_fp32": (lambda: dataclasses.replace(refined(), nx=34, ny=16, nz=17, solid=None), "fp32"),
}


def run(case, dtype, tile):
    s = Solver(case, dtype, tile=tile)
    s.init_maxwellian()
    s.kinetic_step(2)
    return s


@pytest.mark.parametrize("name", list(CASES))
def test_segments(name):
    make, dtype = CASES[name]
    case = make()
    print(name, case.nx, case.ny, case.nz, case.nv, dtype, flush=True)
    esz = 8 if dtype == "fp64" else 4
    assert case.ncell * case.nvel * esz * (2 if case.species == I.DIATOMIC else 1) > 256e6
    s = run(case, dtype, (8, 4, 8, 256) if name.endswith("8x4") else None)
    assert s.get_tile()[3] == 256
    a = s.moments()
    live = np.ones(case.ncell, bool) if case.solid is None else np.asarray(case.solid).reshape(-1) == 0
    if case.velocity_list is None:
        g = node_grid(case)
        xi, w = torch.as_tensor(np.asarray(g[0])).cuda(), torch.as_tensor(np.asarray(g[1])).cuda()
    else:
        nodes = torch.as_tensor(case.velocity_list).cuda()
        xi, w = nodes[:, :3].contiguous(), nodes[:, 3].contiguous()
    f = s.get_vdf()[0]
    if dtype == "fp32":
        f = f.float().double()
    rho = (f @ w).cpu().numpy()
    u = (f @ (w[:, None] * xi)).cpu().numpy() / rho[:, None]
    e = (f @ (w * (xi * xi).sum(1))).cpu().numpy() / rho
    T = (e - (u * u).sum(1)) * 2.0 / 3.0
    assert np.abs(a[live, 0] / rho[live] - 1.0).max() < 1e-12
    # |u|^2 and T are differences of the energy sum
    assert np.abs((a[live, 4] - T[live]) / e[live]).max() < 1e-12
    del f, s
    b = run(case, dtype, (4, 4, 4, 128)).moments()
    assert np.array_equal(a, b, equal_nan=True)


def test_batch():
    cases = [box((5, 9, 3), (60, 60, 60)), box((4, 4, 4), (80, 81, 82)), box((13, 3, 6), (31, 30, 33))]
    b = Batch(cases, "fp64")
    b.init_maxwellian()
    b.run(2, 4)
    for k, c in enumerate(cases):
        s = Solver(c, "fp64", tile=(4, 4, 4, 128))
        s.init_maxwellian()
        for _ in range(2):
            s.kinetic_step()
            s.gsis_correct(4)
        assert np.array_equal(b[k].moments(), s.moments())
