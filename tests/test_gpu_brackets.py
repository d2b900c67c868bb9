"""The status and the evaluation count of a reconstruction that is given a
bracket per cell and a fixed isovalue, where no search runs.  One cell per group
and in teams, against the oracle."""
import numpy as np
import pytest

import oracle
from tests import parity
from tests.test_gpu_teams import V, _case  # noqa: F401  (V is a fixture)

pytestmark = pytest.mark.gpu

PER_CELL = ("mixed_idx", "s", "n", "A", "d", "alpha_got", "status", "iters")
COUNTS = (None, 3000, 900)   # every mixed cell, and two counts at which teams form


def _first(g, m):
    return {k: (v[..., :m] if k in PER_CELL else v) for k, v in g.items()}


def _fixed_iso(V, kind, form, check):  # noqa: F811
    """check(cells listed, results, oracle) of cuts at 0.5 with the bracket
    [0.6, 0.9] or the network's on every cell."""
    import torch
    from paper_2604_14938_amd import runner, train
    wl, _ = _case(kind)
    rec = oracle.reconstruct(wl.mesh, wl.alpha, fixed_iso=True, iso=0.5)
    run = runner.PathRun(wl, ctx=V.Context(0, stream=torch.cuda.Stream()))
    run.step()
    full = run.results()
    b, M = run.buf, full["n_mixed"]
    lo, hi = torch.full((M,), 0.6, dtype=torch.float64, device=run.dev), torch.full((M,), 0.9, dtype=torch.float64,
                                                                                   device=run.dev)
    params, scale, _ = train.load()
    mlp = V.Mlp(run.ctx)
    mlp.set_params(params)
    for m in COUNTS:
        m = m or M
        print(f"[gpu-case] fixed isovalue {kind} {form}: {m} of {M} cells", flush=True)
        cnt = torch.tensor([m, full["n_band"]], dtype=torch.int32, device=run.dev)
        torch.cuda.synchronize()
        if form == "hint":
            V.reconstruct(run.ctx, run.mesh, run.alpha, b.mixed_idx, cnt, b.itf,
                          V.recon_opts(fixed_iso=1, iso=0.5, bracket=V.BRACKET_HINT), lo, hi)
        else:
            V.reconstruct_learned(run.ctx, run.mesh, run.alpha, b.mixed_idx, cnt, b.itf, mlp, scale,
                                  V.recon_opts(fixed_iso=1, iso=0.5))
        torch.cuda.synchronize()
        check(m, _first(run.results(), m), wl, rec)
    run.close()
    mlp.close()


@pytest.mark.parametrize("kind", ["hex", "voronoi"])
@pytest.mark.parametrize("form", ["hint", "network"])
def test_a_fixed_isovalue_is_not_judged_by_the_bracket(V, kind, form):  # noqa: F811
    def check(m, g, wl, rec):
        idx = g["mixed_idx"]
        np.testing.assert_array_equal(g["status"], rec["status"][idx])
        # (some cuts pass within rounding of a vertex: areas of 1e-33, whose
        # normals are the rounding's)
        cut = (rec["A"][idx] == 0) | (rec["A"][idx] > 1e-9 * wl.mesh.h ** 2)
        parity.check_interface(wl, {k: (v[..., cut] if k in PER_CELL else v) for k, v in g.items()}, rec)

    _fixed_iso(V, kind, form, check)


@pytest.mark.parametrize("kind", ["hex", "voronoi"])
def test_a_fixed_isovalue_is_one_evaluation(V, kind):  # noqa: F811
    _fixed_iso(V, kind, "hint",
               lambda m, g, wl, rec: np.testing.assert_array_equal(g["iters"], rec["iters"][g["mixed_idx"]]))
