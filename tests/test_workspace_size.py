"""What the device workspace may hold beyond the VDF: sizes only, no GPU.

Bounds: a second-order context keeps one more array of the VDF's size per VDF
(its right-hand side); everything per cell is at most 2 KB.
"""
import dataclasses

import pytest

from paper_2310_18916_amd import gsis as G
from paper_2310_18916_amd import inputs as I

GAS = {"species": I.DIATOMIC, "dr": I.N2_DR, "Zr": I.N2_ZR, "A": I.N2_A}
CELL = 2048


def box(n, m, **kw):
    c = dataclasses.replace(I.cavity(4, 4, 0.1, lid=0.2), **kw)
    c.nx, c.ny, c.nz, c.nv = *n, m
    return c


def vdf_bytes(case, dtype):
    return case.ncell * case.nvel * (8 if dtype == "fp64" else 4) * (2 if case.species == I.DIATOMIC else 1)


@pytest.mark.parametrize("kw", [{}, GAS])
@pytest.mark.parametrize("dtype", ["fp64", "fp32"])
@pytest.mark.parametrize("n, m", [((12, 11, 10), (12, 12, 12)), ((24, 24, 24), (32, 32, 32)),
                                  ((72, 72, 72), (32, 32, 32))])
def test_second_order_adds_one_array(n, m, dtype, kw):
    case = box(n, m, **kw)
    first = G.Context(case, dtype).workspace_size()
    second = G.Context(dataclasses.replace(case, order=2), dtype).workspace_size()
    assert second - first <= vdf_bytes(case, dtype) * (1 + 1 / case.ncell) + 4096
