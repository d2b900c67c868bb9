"""The gradient of every cell with each number of lanes a cell that its launch
rule takes: one and two lanes on meshes above the rule's 32,768 cells, two and
four below, hexahedra and polyhedra, cell counts that fill no block evenly."""
import numpy as np
import pytest

import oracle
from synth import meshes, workloads
from tests import parity
from tests.test_gpu_extrap import R, _say  # noqa: F401  (R is a fixture)

pytestmark = pytest.mark.gpu

MESHES = {"one": lambda: meshes.hex_mesh(33), "two_hex": lambda: meshes.hex_mesh(13),
          "two": lambda: meshes.voronoi_box_mesh(26, seed=5), "four": lambda: meshes.voronoi_box_mesh(11, seed=5)}


@pytest.mark.parametrize("lanes", sorted(MESHES))
def test_every_cell(R, lanes):  # noqa: F811
    import torch
    from paper_2604_14938_amd import vofpc as V
    wl = workloads.random_bubbles(MESHES[lanes](), seed=8, n_max=6, K=16, r_hi_h=3.0)
    N = wl.mesh.n_cells
    assert (N > 32768) == (lanes in ("one", "two"))
    geom = oracle.geometry(wl.mesh)
    run = R.PathRun(wl)
    run.step()
    cases = [(0, False), (1, False)] + ([(2, True)] if lanes in ("two", "four") else [])
    for weight, extended in cases:
        _say(f"gradient {lanes}: {N} cells, weight {weight}, vertex stencil {extended}")
        out = torch.full((3, N), float("nan"), dtype=torch.float64, device=run.dev)
        st = torch.full((N,), -7, dtype=torch.int32, device=run.dev)
        torch.cuda.synchronize()
        var = V.GRAD_MODIFIED | {0: 0, 1: V.GRAD_W_INV_DIST, 2: V.GRAD_W_INV_DIST2}[weight]
        V.grad_T(run.ctx, run.mesh, run.T, run.Tb, wl.T_sat, run.alpha, None, None, out, st, scope=V.SCOPE_ALL,
                 variant=var | (V.GRAD_VERTEX_STENCIL if extended else 0))
        torch.cuda.synchronize()
        ref, rst = oracle.grad(wl.mesh, geom, wl.T, wl.T_bface, wl.T_sat, wl.alpha, weight=weight, extended=extended)
        parity.check_grad(wl, out.cpu().numpy(), ref, np.arange(N))
        np.testing.assert_array_equal(st.cpu().numpy(), rst)
    run.close()
