"""The built-in sweep tile of boxes so long that 4-cell tiles would be more than
the 1023 that a packed tile index may count: a tile that gsis_set_tile takes too,
for one box and for a batch, and (GPU) the bits of a tile of another shape.

Tolerance: none.  A cell's update has a fixed operand order, so its VDF does not
depend on the tile.
"""
import ctypes as C
import dataclasses

import numpy as np
import pytest

from paper_2310_18916_amd import gsis as G
from paper_2310_18916_amd import inputs as I

GAS = {"species": I.DIATOMIC, "dr": I.N2_DR, "Zr": I.N2_ZR, "A": I.N2_A}
KINDS = [("fp64", {}), ("fp32", {}), ("fp64", GAS), ("fp32", GAS)]


def box(n, m, **kw):
    c = dataclasses.replace(I.cavity(4, 4, 0.1, lid=0.2), **kw)
    c.nx, c.ny, c.nz, c.nv = *n, m
    return c


@pytest.mark.parametrize("dtype, kw", KINDS)
@pytest.mark.parametrize("long", [4092, 4093, 4096])
def test_accepted(long, dtype, kw):
    t, h = (C.c_int * 4)(), C.c_void_p()
    boxes = [tuple(long if a == k else 1 for k in range(3)) for a in range(3)]
    for n in boxes:
        ctx = G.Context(box(n, (4, 4, 4), **kw), dtype)
        assert ctx.L.gsis_get_tile(ctx.h, t) == 0
        assert all(-(-k // s) <= 1023 for k, s in zip(n, t)), (n, tuple(t))
        assert ctx.L.gsis_set_tile(ctx.h, *t) == 0
        ctxs = [G.Context(box(k, (4, 4, 4), **kw), dtype) for k in (n, (8, 8, 8))]
        arr = (C.c_void_p * 2)(*[c.h.value for c in ctxs])
        assert ctx.L.gsis_batch_create(C.byref(h), arr, 2) == 0
        ctx.L.gsis_batch_destroy(h)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype, kw", KINDS)
@pytest.mark.parametrize("n", [(1, 4094, 2), (4095, 2, 1)])
def test_pass_bitwise(n, dtype, kw):
    out = []
    for tile in (None, (8, 4, 8, 128) if n[0] > 1 else (8, 8, 1, 256) if not (kw and dtype == "fp32") else (16, 8, 1, 256)):
        s = G.Solver(box(n, (6, 5, 4), **kw), dtype, tile=tile)
        s.init_maxwellian()
        s.kinetic_step(2)
        out.append((s.moments(), s.get_vdf()[0].cpu().numpy()))
    for a, b in zip(*out):
        assert np.array_equal(a, b)
