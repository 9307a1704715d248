"""A run has the same bits however its steps are taken: in passes of two, one at a time, with a check
between the two steps of a pass, saved and restored at an odd step, or recorded.  Compared are the
populations themselves (of a checkpoint) and the boundary solver's state, on grids that take passes.
"""
import pytest

from test_gpu_pair import CASES, P, RELAX, fields

pytestmark = pytest.mark.gpu
IDS = [f"q{c[0]}-{c[1][0]}x{c[1][1]}-{'_'.join(b[:6] for b in c[2])}-{c[3]}" for c in CASES]


def make(q, size, bc, precision, opts):
    from paper_2307_16766_amd import lbm
    nx, ny = size
    s = lbm.LBM(q, nx, ny, {9: 0.6, 17: 0.9, 37: 0.64}[q], bc, fields(nx, ny, 11), precision=precision)
    s.set_relax(-1, **RELAX)
    if "recon" in opts:
        s.set_reconstruction(-1, opts["recon"])
    if "visc" in opts:
        s.set_viscous(-1, opts["visc"])
    return s


def state(s, q, bc, precision):
    """Populations f[y][i][x] of a checkpoint (behind its 256-byte header; rows padded to 64 values) and
    the boundary state of the characteristic sides."""
    import torch
    pitch = (s.nx + 63) // 64 * 64
    size, kind = (8, torch.float64) if precision == "fp64" else (4, torch.float32)
    f = s.save()[256:256 + q * pitch * s.ny * size].view(kind).reshape(s.ny, q, pitch)[:, :, :s.nx]
    M = 1 if q == 9 else 3
    return [f] + [s.boundary_state(k, M, (s.ny if k < 2 else s.nx) - (2 * M if P not in bc else 0))
                  for k, b in enumerate(bc) if b in ("lodi", "lodi_relax", "cbc", "cbc_relax")]


def same(a, b):
    import torch
    assert len(a) == len(b)
    for u, v in zip(a, b):
        assert torch.equal(u, v)


@pytest.mark.parametrize("q,size,bc,precision,steps,opts", CASES, ids=IDS)
def test_passes_equal_single_steps(q, size, bc, precision, steps, opts):
    a, b = [make(q, size, bc, precision, opts) for _ in range(2)]
    a.step(steps)
    for _ in range(steps):
        b.step(1)
    same(state(a, q, bc, precision), state(b, q, bc, precision))
    a.close()
    b.close()


RUNS = [(37, (1021, 1607), ["lodi_relax", "cbc_relax", "lodi", "cbc"], "fp64", {}),
        (37, (1607, 1021), ["cbc", "lodi_relax", P, P], "fp32dev", dict(recon="neep")),
        (17, (1021, 1607), [P] * 4, "fp64", {}), (9, (1607, 1021), [P, P, "lodi", "zg"], "fp32dev", {})]


@pytest.mark.parametrize("q,size,bc,precision,opts", RUNS, ids=[f"q{r[0]}-{r[3]}" for r in RUNS])
def test_split_checked_restored_and_recorded_runs(q, size, bc, precision, opts):
    n = 7
    ref = make(q, size, bc, precision, opts)
    ref.step(n)
    want = state(ref, q, bc, precision)
    ref.close()
    for at in (1, 4):                       # a run saved and restored there
        s = make(q, size, bc, precision, opts)
        s.step(at)
        buf = s.save()
        s.step(3)
        s.restore(buf)
        s.step(n - at)
        same(state(s, q, bc, precision), want)
        s.close()
    s = make(q, size, bc, precision, opts)  # checks after steps 3 and 6
    s.set_diag_every(3)
    s.step(n)
    same(state(s, q, bc, precision), want)
    s.close()
    s = make(q, size, bc, precision, opts)
    s.record(n, 2)
    same(state(s, q, bc, precision), want)
    s.close()
