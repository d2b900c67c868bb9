"""The sweeps of the extrapolation at the edges of their launch: a domain beyond
the cells that one launch keeps in registers (256 blocks of 256 cells), cells
with more upwind faces than a group keeps, sweep caps of 1 and 2, and two
meshes whose sweeps run at the same time."""
import numpy as np
import pytest

from synth import meshes, workloads
from tests.test_gpu_extrap import R, _oracle, _run, _say  # noqa: F401  (R is a fixture)

pytestmark = pytest.mark.gpu

KEPT_CELLS, KEPT_SLOTS = 256 * 256, 10


def _hex_many(seed=31):
    return workloads.random_bubbles(meshes.hex_mesh(52), seed=seed, n_max=700, K=16, r_hi_h=5.0)


def _undirected(wl):
    """Cells whose neighbours' alphas cancel exactly about them (between two
    bubbles on a uniform grid): the plain gradient is zero but for rounding,
    and so its direction says nothing."""
    m, a = wl.mesh, wl.alpha
    s = np.zeros((3, m.n_cells))
    inner = np.nonzero(m.face_neigh >= 0)[0]
    P, Q = m.face_owner[inner], m.face_neigh[inner]
    c = m.cell_vertex_mean()
    w = (a[Q] - a[P])[:, None] * (c[Q] - c[P])
    for d in range(3):
        np.add.at(s[d], P, w[:, d])
        np.add.at(s[d], Q, w[:, d])
    size = np.zeros(m.n_cells)
    np.add.at(size, P, np.abs(w).sum(1))
    np.add.at(size, Q, np.abs(w).sum(1))
    return (size > 0) & (np.abs(s).max(0) <= 1e-12 * size)


def _check(wl, g, ref, opts):
    assert g["err"] == 0 and g["sweeps"] == ref["sweeps"], (opts, g["sweeps"], ref["sweeps"])
    dom = ref["dom"]
    np.testing.assert_array_equal(~np.isnan(g["gl"][0]), dom)
    scale = np.abs(ref["grad"][:, dom]).max()
    dom = dom & ~_undirected(wl)
    for k in ("gl", "gv"):
        assert np.abs(g[k][:, dom] - ref[k][:, dom]).max() <= 1e-9 * scale, (opts, k)


@pytest.mark.parametrize("case", ["kept_cells", "kept_slots"])
def test_beyond_the_registers(R, case):  # noqa: F811
    if case == "kept_cells":
        wl, runs = _hex_many(), [dict(layers=4), dict(layers=4, max_iter=1), dict(layers=4, max_iter=2)]
    else:
        wl = workloads.random_bubbles(meshes.voronoi_box_mesh(16, seed=32), seed=33, n_max=40, K=16, r_hi_h=3.0)
        runs = [dict(layers=3, tol=1e-6, max_iter=400)]
        # half of a cell's faces are upwind of some direction or of its reverse
        assert np.diff(wl.mesh.cell_face_off).max() > 2 * KEPT_SLOTS
    for opts in runs:
        _say(f"extrapolation {case} {opts}")
        g, ref = _run(R, wl, **opts), _oracle(wl, **opts)
        if case == "kept_cells":
            assert ref["dom"].sum() > KEPT_CELLS
        _check(wl, g, ref, opts)
        g["run"].close()


@pytest.mark.parametrize("captured", [False, True])
def test_two_meshes_at_once(R, captured):  # noqa: F811
    """Each on its own stream, each as large as the chip: issued together,
    eager and from graphs, with the results of one alone."""
    import torch
    from paper_2604_14938_amd import vofpc as V
    opts = dict(layers=4, tol=1e-7, max_iter=60)
    _say(f"extrapolation of two meshes, captured {captured}")
    sides = []
    for seed in (31, 47):
        wl = _hex_many(seed)
        g = _run(R, wl, **opts)
        assert g["err"] == 0
        run, b = g["run"], g["run"].buf
        gl, gv = (torch.zeros(3, wl.mesh.n_cells, dtype=torch.float64, device=run.dev) for _ in range(2))
        rep = torch.zeros(2, dtype=torch.int32, device=run.dev)
        torch.cuda.synchronize()

        def call(run=run, b=b, wl=wl, gl=gl, gv=gv, rep=rep):
            V.extrapolate(run.ctx, run.mesh, run.alpha, run.T, run.Tb, wl.T_sat, b.mixed_idx, b.counts, b.itf, gl, gv,
                          rep, opts=V.extrap_opts(**opts))
        if captured:
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph, stream=run.ctx.stream):
                call()
            call = (lambda graph=graph, s=run.ctx.stream: _replay(graph, s))
        sides.append((g, call, gl, gv, rep))
    for _ in range(3):
        for _g, _c, gl, gv, _r in sides:
            gl.zero_()
            gv.zero_()
        torch.cuda.synchronize()
        for _g, call, *_ in sides:
            call()
        torch.cuda.synchronize()
        for g, _c, gl, gv, rep in sides:
            dom = ~np.isnan(g["gl"][0])
            assert int(rep[1].item()) == 0 and int(rep[0].item()) == g["sweeps"]
            np.testing.assert_array_equal(gl.cpu().numpy()[:, dom], g["gl"][:, dom])
            np.testing.assert_array_equal(gv.cpu().numpy()[:, dom], g["gv"][:, dom])
    for g, *_ in sides:
        g["run"].close()


def _replay(graph, stream):
    import torch
    with torch.cuda.stream(stream):
        graph.replay()
