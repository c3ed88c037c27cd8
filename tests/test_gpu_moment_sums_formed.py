"""Which kernel makes the moment sums: the sweep really forms them in the cases of
test_gpu_moment_segments.py and doesn't in their 128-thread twins nor in an FP32 tile
8 cells wide, and the
compiled variants that those leave out (second order with two VDFs and in FP32, a
per-point term with solid cells and in FP32) give the same bits both ways.

Tolerances: as there (bitwise; 1e-12 of a sum of positive terms against a plain
FP64 product).
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
from test_gpu_moment_segments import CASES, GAS, box, solid  # noqa: E402

WIDTH = {"two_vdfs_wide": 8, "two_vdfs_solid": 4, "solid": 4}


@pytest.mark.parametrize("name", [n for n in CASES if n not in ("few_nodes", "over_fp32_8x4")])
def test_formed(name):
    make, dtype = CASES[name]
    case = make()
    s = Solver(case, dtype)
    assert s.forms_sums()
    assert s.get_tile()[0] == WIDTH.get(name, s.get_tile()[0])
    s.set_tile(4, 4, 4, 128)
    assert not s.forms_sums()


def test_not_formed():
    for name, tile in (("few_nodes", None), ("over_fp32_8x4", (8, 4, 8, 256))):
        make, dtype = CASES[name]
        assert not Solver(make(), dtype, tile=tile).forms_sums()


def test_formed_batch():
    cases = [box((5, 9, 3), (60, 60, 60)), box((4, 4, 4), (80, 81, 82)), box((13, 3, 6), (31, 30, 33))]
    b = Batch(cases, "fp64")
    assert all(m.forms_sums() for m in b.members)


def solid_term(dtype):
    c = solid(I.MONATOMIC)
    return dataclasses.replace(c, inv_dt=3.0, nv=(52, 51, 53) if dtype == "fp32" else c.nv)


MORE = {
    "second_order_two_vdfs": (lambda: box((6, 5, 4), (54, 55, 53), order=2, **GAS), "fp64"),
    "second_order_two_vdfs_fp32": (lambda: box((6, 5, 5), (66, 65, 67), order=2, **GAS), "fp32"),
    "second_order_fp32": (lambda: box((6, 5, 5), (80, 79, 81), order=2), "fp32"),
    "term_fp32": (lambda: box((5, 9, 3), (90, 89, 91), inv_dt=3.0), "fp32"),
    "term_solid": (lambda: solid_term("fp64"), "fp64"),
    "term_solid_fp32": (lambda: solid_term("fp32"), "fp32"),
    "term_two_vdfs": (lambda: box((5, 5, 3), (70, 71, 69), inv_dt=3.0, **GAS), "fp64"),
    "term_two_vdfs_solid": (lambda: dataclasses.replace(solid(I.DIATOMIC), inv_dt=3.0), "fp64"),
}


def run(case, dtype, tile):
    s = Solver(case, dtype, tile=tile)
    s.init_maxwellian()
    s.kinetic_step(2)
    return s


@pytest.mark.parametrize("name", list(MORE))
def test_more(name):
    make, dtype = MORE[name]
    case = make()
    print(name, case.nx, case.ny, case.nz, case.nv, dtype, flush=True)
    s = run(case, dtype, None)
    assert s.forms_sums()
    a = s.moments()
    live = np.ones(case.ncell, bool) if case.solid is None else np.asarray(case.solid).reshape(-1) == 0
    g = node_grid(case)
    xi, w = torch.as_tensor(np.asarray(g[0])).cuda(), torch.as_tensor(np.asarray(g[1])).cuda()
    f = s.get_vdf()[0]
    rho = (f @ w).cpu().numpy()[live]
    e = (f @ (w * (xi * xi).sum(1))).cpu().numpy()[live] / rho
    u = (f @ (w[:, None] * xi)).cpu().numpy()[live] / rho[:, None]
    assert np.abs(a[live, 0] / rho - 1.0).max() < 1e-12
    assert np.abs((a[live, 4] - (e - (u * u).sum(1)) * 2.0 / 3.0) / e).max() < 1e-12
    del f, s
    t = run(case, dtype, (4, 4, 4, 128))
    assert not t.forms_sums()
    assert np.array_equal(a, t.moments(), equal_nan=True)
