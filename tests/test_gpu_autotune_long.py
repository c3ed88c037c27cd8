"""The autotuners on boxes so long that some of their configurations would be more
tiles than a packed tile index counts (1023 per axis): those are left out, and the
pass is a plain one.

Tolerance: none.
"""
import dataclasses

import numpy as np
import pytest

from paper_2310_18916_amd import inputs as I

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2310_18916_amd.gsis import Batch, Solver  # noqa: E402


def box(n, m):
    c = dataclasses.replace(I.cavity(4, 4, 0.1, lid=0.2))
    c.nx, c.ny, c.nz, c.nv = *n, m
    return c


def plain(case, dtype, passes):
    s = Solver(case, dtype)
    s.init_maxwellian()
    s.kinetic_step(passes)
    return s.moments()


def fits(n, table):
    return all(-(-k // s) <= 1023 for (t, _) in table for k, s in zip(n, t))


@pytest.mark.parametrize("dtype", ["fp64", "fp32"])
@pytest.mark.parametrize("n", [(2, 1, 4096), (1, 4095, 2)])
def test_long(n, dtype):
    case = box(n, (5, 4, 6))
    s = Solver(case, dtype)
    s.init_maxwellian()
    table = s.autotune(reps=1)
    assert table and fits(n, table)
    s.kinetic_step(1)
    assert np.array_equal(s.moments(), plain(case, dtype, 2))


def test_long_batch():
    cases = [box((2, 1, 2100), (5, 4, 6)), box((9, 5, 7), (6, 6, 6))]
    b = Batch(cases, "fp32")
    b.init_maxwellian()
    table = b.autotune(reps=1)
    assert table and fits((2, 1, 2100), table)
    for k, c in enumerate(cases):
        assert np.array_equal(b[k].moments(), plain(c, "fp32", 1))
