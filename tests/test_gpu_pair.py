"""Two steps per pass over memory: step(n) on grids large enough for the pass against the same run
advanced one step at a time (the single-step kernel, which the parity tests compare with the oracle).

Both take the same map with the same arithmetic per node, so they differ by rounding only: the
tolerances are those of the parity tests (1e-12 in FP64, 2e-5 in FP32 deviation storage, relative
L2 error of each field).  The sizes are no multiples of the tiles, the step counts even and odd;
every boundary kind, with corners and along both axes.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

TALL, WIDE = (1021, 5407), (5407, 1021)
RELAX = dict(sigma=0.25, alpha=0.1, mach=0.1)


def fields(nx, ny, seed):
    import torch
    g = torch.Generator(device="cuda").manual_seed(seed)

    def waves(a):
        k = torch.rand(4, generator=g, device="cuda", dtype=torch.float64) * 0.05
        x = torch.arange(nx, device="cuda", dtype=torch.float64)[None, :]
        y = torch.arange(ny, device="cuda", dtype=torch.float64)[:, None]
        return a * (torch.sin(k[0] * x + k[1] * y + 10 * k[2])
                    + 0.2 * torch.randn(ny, nx, generator=g, device="cuda", dtype=torch.float64))

    return 1 + waves(1e-3), 0.03 + waves(1e-2), 0.02 + waves(1e-2), 1 + waves(1e-3)


P = "periodic"
CASES = [
    (37, TALL, [P] * 4, "fp64", 4, {}),
    (37, TALL, [P] * 4, "fp32dev", 3, {}),
    (37, (701, 503), [P] * 4, "fp64", 4, {}),          # the shortest row segments
    (9, (1023, 701), [P] * 4, "fp32dev", 4, {}),
    (37, WIDE, ["lodi_relax", "cbc_relax", P, P], "fp64", 5, {}),
    (37, WIDE, ["cbc", "lodi", P, P], "fp32dev", 4, dict(recon="neep")),
    (37, TALL, [P, P, "cbc_relax", "lodi_relax"], "fp64", 4, dict(recon="neep")),
    (37, WIDE, [P, P, "lodi", "cbc_relax"], "fp32dev", 5, dict(visc="fd")),
    (37, TALL, ["lodi_relax"] * 4, "fp64", 5, {}),
    (37, WIDE, ["lodi_relax", "lodi", "cbc_relax", "lodi_relax"], "fp32dev", 4, {}),
    (37, TALL, ["zg"] * 4, "fp64", 4, {}),
    (37, WIDE, ["dirichlet", "lodi_relax", P, P], "fp32dev", 6, {}),
    (37, TALL, [P, P, "zg", "dirichlet"], "fp64", 5, {}),
    (17, TALL, [P] * 4, "fp64", 5, {}),
    (17, WIDE, ["lodi_relax"] * 4, "fp32dev", 4, {}),
    (17, TALL, ["dirichlet", "cbc_relax", P, P], "fp64", 4, {}),
    (9, TALL, [P] * 4, "fp32dev", 5, {}),
    (9, WIDE, ["lodi_relax"] * 4, "fp64", 4, dict(recon="neep")),
    (9, TALL, [P, P, "dirichlet", "lodi_relax"], "fp64", 5, {}),
    (9, WIDE, ["zg", "lodi", P, P], "fp32dev", 4, {}),
]


@pytest.mark.parametrize("q,size,bc,precision,steps,opts", CASES,
                         ids=[f"q{c[0]}-{c[1][0]}x{c[1][1]}-{'_'.join(b[:6] for b in c[2])}-{c[3]}" for c in CASES])
def test_two_steps_per_pass_equal_single_steps(q, size, bc, precision, steps, opts):
    import torch
    from paper_2307_16766_amd import lbm
    nx, ny = size
    f = fields(nx, ny, 11)
    tau = {9: 0.6, 17: 0.9, 37: 0.5 + 0.1 / lbm.lattice_info(37)[0]}[q]
    sims = [lbm.LBM(q, nx, ny, tau, bc, f, precision=precision) for _ in range(2)]
    for s in sims:
        s.set_relax(-1, **RELAX)
        if "recon" in opts:
            s.set_reconstruction(-1, opts["recon"])
        if "visc" in opts:
            s.set_viscous(-1, opts["visc"])
    sims[0].step(steps)
    for _ in range(steps):
        sims[1].step(1)
    assert sims[0].steps_done() == sims[1].steps_done() == steps
    tol = 1e-12 if precision == "fp64" else 2e-5
    a, b = [s.macroscopic() for s in sims]
    for k in range(4):
        err = float((a[k] - b[k]).norm() / b[k].norm())
        assert np.isfinite(err) and err <= tol, (k, err)
    M = 1 if q == 9 else 3
    for side, kind in enumerate(bc):   # the boundary solver's own state
        if kind in ("lodi", "lodi_relax", "cbc", "cbc_relax"):
            corners = P not in bc
            length = (ny if side < 2 else nx) - (2 * M if corners else 0)
            ub, vb = [s.boundary_state(side, M, length) for s in sims]
            err = float((ub - vb).norm() / vb.norm())
            assert np.isfinite(err) and err <= tol, (side, err)
    # layers and corners node by node, not only in the whole field's norm
    for k in range(4):
        d = (a[k] - b[k]).abs()
        edge = torch.cat([d[:6].flatten(), d[-6:].flatten(), d[:, :6].flatten(), d[:, -6:].flatten()])
        assert float(edge.max()) <= 50 * tol * float(b[k].abs().max()), k
    for s in sims:
        s.close()


def test_non_finite_check_between_paired_steps():
    """A check interval that falls between two steps of a pass is kept, and timing counts every step."""
    from paper_2307_16766_amd import lbm
    nx, ny = TALL
    f = fields(nx, ny, 5)
    s = lbm.LBM(37, nx, ny, 0.7, ["lodi_relax", "cbc_relax", P, P], f)
    s.set_relax(-1, **RELAX)
    s.set_diag_every(3)
    s.set_kernel_timing(True, every=3)
    s.step(7)
    assert s.steps_done() == 7
    ms, n = s.bulk_kernel_time()
    assert n == 3 and ms > 0.0          # steps 0, 3 and 6
    s.step(0)
    s.set_diag_every(0)
    bad = f[0].clone()
    bad[ny // 2, nx // 2] = float("nan")
    t = lbm.LBM(37, nx, ny, 0.7, [P] * 4, (bad, *f[1:]))
    t.set_diag_every(5)
    with pytest.raises(lbm.LBMError) as e:
        t.step(8)
    assert e.value.code == lbm.LBM_E_NONFINITE and t.steps_done() == 5
    s.close()
    t.close()
