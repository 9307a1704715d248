"""A recorded run keeps its last two segments for the reverse sweep.  The recording advances the state
exactly as step() does, bit by bit, whatever the segments; and the sweep over kept segments equals
the sweep that recomputes them (a second adjoint() of the same recording), up to nothing: both read
the values that the same kernel wrote.
"""
import pytest

pytestmark = pytest.mark.gpu
P = "periodic"


@pytest.mark.parametrize("steps,every", [(1, 50), (5, 5), (6, 5), (11, 5), (23, 5)])
@pytest.mark.parametrize("q,bc,precision", [
    (37, ["lodi_relax"] * 4, "fp64"), (37, ["cbc_relax", "cbc", "cbc_relax", "lodi_relax"], "fp64"),
    (17, ["cbc_relax"] * 4, "fp32dev"), (9, ["lodi", "zg", P, P], "fp64"), (37, [P, P, "dirichlet", "lodi_relax"], "fp64"),
    (37, [P] * 4, "fp32dev")])
def test_recorded_segments(q, bc, precision, steps, every):
    import torch
    from paper_2307_16766_amd import lbm
    nx, ny = 61, 47
    g = torch.Generator(device="cuda").manual_seed(3)

    def noise(a):
        return a * torch.rand(ny, nx, generator=g, device="cuda", dtype=torch.float64)

    f = (1 + noise(1e-3), 0.03 + noise(1e-2), 0.02 + noise(1e-2), 1 + noise(1e-3))
    plain, rec = [lbm.LBM(q, nx, ny, 0.7, bc, f, precision=precision) for _ in range(2)]
    for s in (plain, rec):
        s.set_relax(-1, sigma=0.25, alpha=0.1, mach=0.1)
    rec.set_kernel_timing(True, every=1)
    plain.step(steps)
    rec.record(steps, every)
    assert rec.steps_done() == steps and rec.bulk_kernel_time()[1] == steps
    first = rec.adjoint()
    again = rec.adjoint()
    assert torch.equal(first[0], again[0]) and (first[1] == again[1]).all()
    for extra in (0, 1, 2):          # the state goes on from the recording as from plain steps
        plain.step(extra)
        rec.step(extra)
        assert torch.equal(torch.stack(plain.macroscopic()), torch.stack(rec.macroscopic()))
    for s in (plain, rec):
        s.close()
