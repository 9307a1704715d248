"""The FP32 collision (pairs of opposite velocities) against the FP64 one, and its invariants.

Fields: the parity tolerance of FP32 deviation storage, 2e-5 (relative L2).  Mass and momentum of a
periodic box: a step rounds each population once (2^-24 of its deviation) and the projection leaves a
residual of the same size, so n steps move a sum over the box by at most 2 n 2^-24 sum |c| |d|.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("amp", [1e-4, 0.08])
@pytest.mark.parametrize("q", [9, 17, 37])
def test_fp32_collision(q, amp):
    import torch
    from paper_2307_16766_amd import lbm
    nx, ny, n = 131, 67, 40
    x = 2 * np.pi * torch.arange(nx, dtype=torch.float64, device="cuda")[None, :] / nx
    y = 2 * np.pi * torch.arange(ny, dtype=torch.float64, device="cuda")[:, None] / ny
    one = torch.ones(ny, nx, dtype=torch.float64, device="cuda")
    f = (one + 1e-3 * torch.sin(x + y), amp * torch.sin(2 * y) + 0.5 * amp * one, amp * torch.cos(x + 2 * y),
         one + (0 if q == 9 else 1e-3) * torch.cos(x - y))
    out, first = {}, {}
    for precision in ("fp32dev", "fp64"):
        s = lbm.LBM(q, nx, ny, 0.7, ["periodic"] * 4, f, precision=precision)
        first[precision] = [v.clone() for v in s.macroscopic()]
        s.step(n)
        out[precision] = s.macroscopic()
        s.close()
    for a, b in zip(out["fp32dev"][:3 if q == 9 else 4], out["fp64"]):
        assert float((a - b).norm() / b.norm()) <= 2e-5
    bound = 2 * n * 2.0 ** -24 * nx * ny * max(2 * amp, 4e-3) * 4     # sum_i |c| |d| <= 4 (rho |u| + |rho - 1| + ..)
    (r0, u0, v0, _), (r1, u1, v1, _) = first["fp32dev"], out["fp32dev"]
    assert abs(float((r1 - r0).sum())) <= bound
    assert abs(float((r1 * u1 - r0 * u0).sum())) <= bound
    assert abs(float((r1 * v1 - r0 * v0).sum())) <= bound
