"""The group reconstruction kernel over the counts at which its schedule
changes: one cell per wavefront (teams of 16 or 4 groups), a quarter of a
wavefront per cell, and full wavefronts; and the large cells of a Voronoi mesh
in the launch of the usual ones and in one of their own.  Compared with the
oracle to the parity bar."""
import numpy as np
import pytest

import oracle
from synth import meshes, workloads
from tests import parity

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def V():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2604_14938_amd import vofpc
    return vofpc


_CASES = {}


def _case(kind):
    if kind not in _CASES:
        mesh = meshes.hex_mesh(72) if kind == "hex" else meshes.voronoi_box_mesh(36, seed=52)
        wl = workloads.random_bubbles(mesh, seed=53, n_max=40, K=10, r_hi_h=9.0)
        _CASES[kind] = (wl, oracle.reconstruct(wl.mesh, wl.alpha))
    return _CASES[kind]


# a launch has at most 8 wavefronts on each of 256 CUs: teams end at twice
# (hexahedra: eight times, in teams of four) that many cells
@pytest.mark.parametrize("kind,tune,learned", [("hex", None, False), ("hex", None, True), ("voronoi", None, False),
                                               ("voronoi", None, True), ("voronoi", (14, 26, 3, 3), False),
                                               ("voronoi", (3, 3, 26, 3), True)])
def test_schedules_match_the_oracle(V, kind, tune, learned):
    import torch
    from paper_2604_14938_amd import runner, train
    wl, rec = _case(kind)
    print(f"[gpu-case] teams {kind} {tune} learned={learned}: {wl.n_mixed} mixed", flush=True)
    ctx = V.Context(0, stream=torch.cuda.Stream())
    mlp, scale = None, 0.0
    if learned:
        params, scale, _ = train.load()
        mlp = V.Mlp(ctx)
        mlp.set_params(params)
    run = runner.PathRun(wl, ctx=ctx, mlp=mlp, delta_scale=scale)
    if tune is not None:
        run.mesh.set_tune(list(tune))
    assert wl.n_mixed > 16384 if kind == "hex" else wl.n_mixed > 4096
    run.step()
    full = run.results()
    b, M = run.buf, full["n_mixed"]
    flags = None
    for m in (M, 16384, 8193, 4097, 4096, 2049, 7, 1):
        if m > M:
            continue
        cnt = torch.tensor([m, full["n_band"]], dtype=torch.int32, device=run.dev)
        b.itf.status.fill_(-1)
        torch.cuda.synchronize()
        if learned:
            V.reconstruct_learned(ctx, run.mesh, run.alpha, b.mixed_idx, cnt, b.itf, mlp, scale)
        else:
            V.reconstruct(ctx, run.mesh, run.alpha, b.mixed_idx, cnt, b.itf)
        g = run.results()
        assert (b.itf.status[m:] == -1).all()
        g = {k: (v[..., :m] if k in ("mixed_idx", "s", "n", "A", "d", "alpha_got", "status", "iters") else v)
             for k, v in g.items()}
        if learned:
            # the brackets, and with them the flags, do not depend on the schedule
            st = g["status"].copy()
            flags = st if flags is None else flags
            np.testing.assert_array_equal(st, flags[:m])
            g["status"] = np.where(st == V.CELL_LEARNED_FALLBACK, V.CELL_OK, st)
        parity.check_interface(wl, g, rec)
    run.close()
    if mlp is not None:
        mlp.close()
