"""One D2Q9 step in FP32 deviation storage against the same operations in numpy, bit for bit: which
products are fused with the sums they enter is part of the source (inside expressions, always).  Rounding
b / cs before it is added to the pair's even part, instead of fusing it, makes the errors against 64
bits 8 % larger.

A fused multiply-add in float32 is taken in float64, where the product is exact, and rounded once more:
that differs from one rounding with a probability of about 2^-29 per operation, so at most one value in
1e5 may differ, by one unit in the last place.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
F = np.float32


def fma(a, b, c):
    return (np.asarray(a, np.float64) * np.asarray(b, np.float64) + np.asarray(c, np.float64)).astype(F)


def collide_d2q9(d, cx, cy, w, omega):
    """Pulled deviations d[9] (pairs p, p + 4) -> post-collision, in float32."""
    s0, jx, jy = d[0], F(0), F(0)
    for p in range(1, 5):
        s0 = s0 + (d[p] + d[p + 4])
        jx, jy = jx + F(cx[p]) * (d[p] - d[p + 4]), jy + F(cy[p]) * (d[p] - d[p + 4])
    rho = F(1) + s0
    ir = F(1) / rho
    ics, cs2 = F(np.sqrt(3.0)), 1.0 / 3.0
    vx, vy = (jx * ir) * ics, (jy * ir) * ics
    u2 = fma(vx, vx, vy * vy)
    C0 = F(-0.5) * u2
    x = [fma(F(w[0]), fma(rho, C0, s0), -d[0])] + [None] * 8
    even = {1: F(0), 2: F(0)}
    mx = my = F(0)
    for p in range(1, 5):
        b = F(cx[p]) * vx + F(cy[p]) * vy
        a = b * ics
        E = fma(F(0.5), a * a, C0)
        x[p] = fma(F(w[p]), fma(rho, fma(b, ics, E), s0), -d[p])
        x[p + 4] = fma(F(w[p]), fma(rho, fma(-b, ics, E), s0), -d[p + 4])
        o, g = x[p] - x[p + 4], int(cx[p] ** 2 + cy[p] ** 2)
        even[g] = even[g] + (x[p] + x[p + 4])
        mx, my = mx + F(cx[p]) * o, my + F(cy[p]) * o
    m0 = (x[0] + even[1]) + even[2]
    a0, a1, a2 = omega * m0, (omega * mx) * F(1 / cs2), (omega * my) * F(1 / cs2)
    out = [d[0] + fma(omega, x[0], -(F(w[0]) * a0))]
    for s in (1, -1):
        for p in range(1, 5):
            hi = F(w[p]) * a0
            if cx[p]:
                hi = hi + F(s * cx[p]) * (F(w[p]) * a1)
            if cy[p]:
                hi = hi + F(s * cy[p]) * (F(w[p]) * a2)
            i = p if s == 1 else p + 4
            out.append(d[i] + fma(omega, x[i], -hi))
    return np.array(out)


def test_d2q9_fp32_step():
    from paper_2307_16766_amd import lbm
    cs2, w, cx, cy, _ = lbm.lattice_info(9)
    cx, cy = cx.astype(int), cy.astype(int)
    nx, ny, tau = 320, 199, 0.7
    rng = np.random.default_rng(3)
    f = (1 + 1e-2 * rng.random((ny, nx)), 0.05 * rng.standard_normal((ny, nx)), 0.05 * rng.standard_normal((ny, nx)), 1.0)
    s = lbm.LBM(9, nx, ny, tau, ["periodic"] * 4, f, precision="fp32dev")

    def populations():
        buf = s.save().cpu().numpy()[256:256 + 9 * nx * ny * 4]
        return buf.view(F).reshape(ny, 9, nx).transpose(1, 0, 2)

    d = populations()
    s.step(1)
    got = populations()
    s.close()
    pulled = [np.roll(d[i], (cy[i], cx[i]), (0, 1)) for i in range(9)]
    want = collide_d2q9(pulled, cx, cy, w, F(1 / tau))
    bad = got != want
    assert bad.sum() <= got.size / 1e5
    assert (np.abs(got[bad] - want[bad]) <= 2 * np.spacing(np.abs(want[bad]))).all()
