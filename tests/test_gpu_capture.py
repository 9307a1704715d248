"""Captured calls on grids where step() takes passes of two steps: a graph of an even number of steps
advances the state at every replay, also mixed with eager calls of an even number of steps and after a
restore, and a graph of macroscopic() reads the state that such calls leave.

Every state is compared with the run taken one step at a time; the tolerances are those of the parity
tests (relative L2 error 1e-12 in FP64, 2e-5 in FP32 deviation storage), and one replay moves u_x by more
than a hundred times that.
"""
import pytest

pytestmark = pytest.mark.gpu
P = "periodic"


@pytest.mark.parametrize("q,size,bc,precision,n", [
    (37, (701, 503), [P] * 4, "fp64", 2), (37, (701, 503), [P] * 4, "fp64", 4), (17, (1021, 1703), [P] * 4, "fp32dev", 6),
    (37, (1021, 1103), ["lodi_relax", "cbc_relax", "lodi_relax", "lodi"], "fp64", 2),
    (9, (1021, 1703), [P, P, "lodi_relax", "dirichlet"], "fp32dev", 2),
    (37, (64, 48), ["lodi_relax"] * 4, "fp64", 2)])   # single steps
def test_replayed_steps(q, size, bc, precision, n):
    import torch
    from paper_2307_16766_amd import lbm
    nx, ny = size
    tol = 1e-12 if precision == "fp64" else 2e-5
    x = torch.arange(nx, device="cuda", dtype=torch.float64)[None, :] / nx
    y = torch.arange(ny, device="cuda", dtype=torch.float64)[:, None] / ny
    wave = torch.sin(6.283185307179586 * (9 * x + 7 * y))
    f = (1 + 0.02 * wave, 0.03 + 0.05 * wave, 0.02 - 0.05 * wave, 1 + 0.01 * wave)
    stream = torch.cuda.Stream()
    stream.wait_stream(torch.cuda.current_stream())
    torch.cuda.synchronize()
    with torch.cuda.stream(stream):
        sim, ref = [lbm.LBM(q, nx, ny, 0.7, bc, f, precision=precision, stream=stream) for _ in range(2)]
        for s in (sim, ref):
            s.set_relax(-1, sigma=0.25, alpha=0.1, mach=0.1)

        def expect(steps, fields):
            before = ref.macroscopic()[1] if steps else None
            for _ in range(steps):
                ref.step(1)
            want = ref.macroscopic()
            torch.cuda.synchronize()
            if steps:
                assert float((want[1] - before).norm() / want[1].norm()) > 100 * tol
            for a, b in zip(fields, want):
                assert float((a - b).norm() / b.norm()) <= tol

        sim.step(10)
        expect(10, sim.macroscopic())
        saved, saved_ref = sim.save(), ref.save()
        graph, look = torch.cuda.CUDAGraph(), torch.cuda.CUDAGraph()
        torch.cuda.synchronize()
        with torch.cuda.graph(graph, stream=stream):
            sim.step(n)
        with torch.cuda.graph(look, stream=stream):
            seen = sim.macroscopic()
        for eager in (0, 2, 6, 0):
            sim.step(eager)
            look.replay()
            expect(eager, seen)
            graph.replay()
            expect(n, sim.macroscopic())
            look.replay()
            expect(0, seen)
        sim.restore(saved)
        ref.restore(saved_ref)
        graph.replay()
        expect(n, sim.macroscopic())
        torch.cuda.synchronize()
        del graph, look
        sim.close()
        ref.close()
