"""The extrapolation while another stream's products hold the compute units: its
blocks come late and take part as they come, and every bit is that of a run on
an idle chip (a Jacobi sweep does not depend on who does it)."""
import pytest

from tests.test_gpu_teams import V, _case  # noqa: F401  (V is a fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("size", [1024, 2048, 4096])
def test_late_blocks_change_no_bit(V, size):  # noqa: F811
    import torch
    from paper_2604_14938_amd import runner
    wl, _ = _case("hex")
    run = runner.PathRun(wl, ctx=V.Context(0, stream=torch.cuda.Stream()))
    run.step()
    b, N = run.buf, wl.mesh.n_cells
    side = torch.cuda.Stream()
    a = torch.ones(size, size, dtype=torch.float64, device=run.dev)
    c = torch.empty_like(a)

    def extrapolate():
        out = [torch.zeros(3, N, dtype=torch.float64, device=run.dev) for _ in range(2)]
        rep = torch.full((2,), 7, dtype=torch.int32, device=run.dev)
        torch.cuda.synchronize()
        return out + [rep], lambda: V.extrapolate(run.ctx, run.mesh, run.alpha, run.T, run.Tb, wl.T_sat, b.mixed_idx,
                                                  b.counts, b.itf, *out, rep)

    quiet, go = extrapolate()
    go()
    torch.cuda.synchronize()
    assert int(quiet[2][0]) > 5 and int(quiet[2][1]) == 0
    for k in range(4):
        print(f"[gpu-case] extrapolation beside products of {size}: {k}", flush=True)
        busy, go = extrapolate()
        with torch.cuda.stream(side):
            for _ in range(k + 1):
                torch.mm(a, a, out=c)
        go()
        torch.cuda.synchronize()
        for x, y in zip(busy, quiet):
            assert torch.equal(x, y)
    run.close()
