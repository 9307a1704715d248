"""Passes of two steps on the narrowest grids that take them: bands that nearly meet, boxes narrower than
a tile (most columns idle, layers of both sides in one tile), one column in the last tile, one short
segment of all rows.  Populations and boundary state against single steps, bit for bit.
"""
import pytest

from test_gpu_pair import P
from test_gpu_same_bits import make, same, state

pytestmark = pytest.mark.gpu

SHAPES = [(9, (12, 8000), [P] * 4, "fp64"), (9, (12, 8001), [P] * 4, "fp32dev"), (9, (249, 3001), [P] * 4, "fp64"),
          (9, (130201, 13), [P] * 4, "fp64"), (37, (30721, 25), [P] * 4, "fp64"), (17, (90, 6001), [P] * 4, "fp64"),
          (37, (64, 5001), [P] * 4, "fp64"), (37, (121, 2001), [P] * 4, "fp64"), (37, (141, 5001), [P] * 4, "fp32dev"),
          (9, (230, 7001), ["lodi", "lodi_relax", "lodi", "lodi"], "fp64"), (9, (230, 6001), ["lodi", "lodi_relax", P, P], "fp64"),
          (9, (24001, 38), [P, P, "lodi", "lodi_relax"], "fp64"), (9, (24001, 40), ["lodi"] * 4, "fp64"),
          (37, (110, 12001), ["dirichlet", "zg", P, P], "fp64"), (37, (61443, 50), ["zg"] * 4, "fp32dev"),
          (17, (220, 9001), ["zg"] * 4, "fp64")]


@pytest.mark.parametrize("q,size,bc,precision", SHAPES, ids=[f"q{s[0]}-{s[1][0]}x{s[1][1]}-{s[2][0]}-{s[3]}" for s in SHAPES])
def test_narrow_grids(q, size, bc, precision):
    import torch
    from paper_2307_16766_amd import lbm
    assert lbm.steps_per_pass(lbm.make_config(q, *size, 0.7, bc, precision)) == 2
    a, b = [make(q, size, bc, precision, {}) for _ in range(2)]
    a.step(6)
    for _ in range(6):
        b.step(1)
    got = state(a, q, bc, precision)
    assert bool(torch.isfinite(got[0]).all())
    same(got, state(b, q, bc, precision))
    a.close()
    b.close()
