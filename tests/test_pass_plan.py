"""Where lbm_step takes two steps per pass (lbm_steps_per_pass): no GPU needed.

The narrow boxes are ones on which a pass was measured slower than two single steps (most of a tile's
columns idle, few rows per segment, or more boundary work than the saved traffic pays for); the others
were measured faster.
"""
import pytest

from paper_2307_16766_amd import lbm
from test_gpu_pair import CASES
from test_gpu_pass_shapes import SHAPES
from test_gpu_same_bits import RUNS

P = "periodic"
X, XY = ["lodi_relax", "cbc_relax", P, P], ["lodi_relax", "cbc_relax", "lodi_relax", "lodi"]
Y = [P, P, "lodi_relax", "lodi"]


def steps(q, size, bc, precision):
    return lbm.steps_per_pass(lbm.make_config(q, *size, 0.7, bc, precision))


@pytest.mark.parametrize("q,size,bc,precision", [
    (37, (24, 3000), [P] * 4, "fp32dev"), (37, (64, 8000), [P] * 4, "fp32dev"), (37, (125, 3000), [P] * 4, "fp32dev"),
    (37, (241, 1300), [P] * 4, "fp32dev"), (37, (40, 8000), [P] * 4, "fp64"), (37, (121, 1300), [P] * 4, "fp64"),
    (37, (125, 1300), [P] * 4, "fp64"), (17, (64, 8000), [P] * 4, "fp64"), (17, (40, 3000), [P] * 4, "fp64"),
    (17, (64, 8000), [P] * 4, "fp32dev"),
    (37, (24, 33784), Y, "fp64"), (37, (100, 8109), X, "fp64"), (37, (33784, 24), XY, "fp64"),
    (37, (24, 99100), Y, "fp32dev"), (37, (250, 9514), X, "fp32dev"), (37, (99100, 24), Y, "fp32dev"),
    (17, (64, 14063), Y, "fp64"), (17, (37501, 24), Y, "fp64"), (17, (1651, 1500), XY, "fp32dev"),
    (17, (161765, 24), Y, "fp32dev"), (9, (64931, 24), Y, "fp32dev"),
    (37, (631, 938), ["zg"] * 4, "fp64"), (37, (592, 880), ["dirichlet", "zg", P, P], "fp64"),
    (37, (1186, 1315), ["zg"] * 4, "fp32dev"), (17, (2139, 466), ["zg"] * 4, "fp64"),
    (37, (702, 768), [P, P, "dirichlet", "cbc"], "fp64"), (37, (622, 822), ["cbc_relax", "cbc_relax", P, P], "fp64")])
def test_single_steps_where_passes_are_slower(q, size, bc, precision):
    if q == 9:
        bc = [b.replace("cbc", "lodi") for b in bc]
    assert steps(q, size, bc, precision) == 1


@pytest.mark.parametrize("q,size,bc,precision", [
    (37, (4096, 2048), X, "fp32dev"), (37, (4096, 2048), XY, "fp64"), (37, (8192, 8192), XY, "fp64"),
    (37, (1023, 509), XY, "fp64"), (37, (2047, 1301), Y, "fp64"), (17, (1950, 1950), [P] * 4, "fp64"),
    (37, (700, 500), [P] * 4, "fp64"), (37, (1024, 512), [P] * 4, "fp32dev"), (9, (12, 8000), [P] * 4, "fp64"),
    (17, (4096, 2048), X, "fp32dev"), (9, (2048, 2048), ["lodi"] * 4, "fp32dev")])
def test_passes_where_they_are_faster(q, size, bc, precision):
    assert steps(q, size, bc, precision) == 2


@pytest.mark.parametrize("q,size,bc,precision", [c[:4] for c in CASES + RUNS + SHAPES])
def test_compared_grids_take_passes(q, size, bc, precision):
    """The comparisons of passes with single steps are on grids that take passes."""
    assert steps(q, size, bc, precision) == 2


def test_invalid_configuration():
    assert steps(37, (64, 48), [P, "lodi", P, P], "fp64") == 0
