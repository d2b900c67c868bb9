"""The isovalue search where its steps change: fractions whose stopping window
is below the rounding of the volume, next to 0 and 1 and in between, one cell per
group and in teams, and narrowed brackets that hold the root and that do not."""
import dataclasses

import numpy as np
import pytest

import oracle
from tests import parity
from tests.test_gpu_teams import V, _case  # noqa: F401  (V is a fixture)

pytestmark = pytest.mark.gpu

PER_CELL = ("mixed_idx", "s", "n", "A", "d", "alpha_got", "status", "iters")
SMALL = np.array([1.1e-8, 1e-6, 1e-4, 1e-3])


@pytest.mark.parametrize("kind", ["hex", "voronoi"])
def test_extreme_fractions(V, kind):  # noqa: F811
    import torch
    from paper_2604_14938_amd import runner
    base, _ = _case(kind)
    alpha = base.alpha.copy()
    rng = np.random.default_rng(3)
    low, high = np.nonzero((alpha > 1e-8) & (alpha < 0.03))[0], np.nonzero((alpha > 0.97) & (alpha < 1 - 1e-8))[0]
    alpha[low], alpha[high] = rng.choice(SMALL, size=low.size), 1.0 - rng.choice(SMALL, size=high.size)
    wl = dataclasses.replace(base, alpha=alpha)
    rec = oracle.reconstruct(wl.mesh, wl.alpha)
    run = runner.PathRun(wl, ctx=V.Context(0, stream=torch.cuda.Stream()))
    run.step()
    full = run.results()
    b, M = run.buf, full["n_mixed"]
    for m in (M, 900):
        print(f"[gpu-case] search {kind}: {m} of {M} cells", flush=True)
        cnt = torch.tensor([m, full["n_band"]], dtype=torch.int32, device=run.dev)
        torch.cuda.synchronize()
        V.reconstruct(run.ctx, run.mesh, run.alpha, b.mixed_idx, cnt, b.itf)
        torch.cuda.synchronize()
        g = run.results()
        g = {k: (v[..., :m] if k in PER_CELL else v) for k, v in g.items()}
        # next to 1 the volume resolves 1 - alpha no finer than 2^-53, and with it
        # the place of a cut of a few parts in 1e8: there the flag and the window
        # are compared, elsewhere everything
        fine = 2.0 ** -53 <= 1e-11 * (1.0 - wl.alpha[g["mixed_idx"]])
        np.testing.assert_array_equal(g["status"], rec["status"][g["mixed_idx"]])
        np.testing.assert_allclose(g["alpha_got"], rec["alpha_got"][g["mixed_idx"]], rtol=0, atol=1e-10)
        parity.check_interface(wl, {k: (v[..., fine] if k in PER_CELL else v) for k, v in g.items()}, rec)
        # a halving search takes some 50 cuts (a team's step counts as 4 or 2) to the adjacent doubles
        assert g["iters"].max() <= 48, np.sort(g["iters"])[-8:]
    run.close()


@pytest.mark.parametrize("shift", [0.0, 0.004, 0.3])
def test_narrowed_brackets(V, shift):  # noqa: F811
    """Brackets about the known isovalue, about a value near it and away from
    it: the isovalue found is the same, and the flag says whether the bracket
    held it."""
    import torch
    from paper_2604_14938_amd import runner, train
    wl, _ = _case("hex")
    params, scale, _ = train.load()
    run = runner.PathRun(wl, ctx=V.Context(0, stream=torch.cuda.Stream()))
    run.step()
    plain = run.results()
    mlp = V.Mlp(run.ctx)
    mlp.set_params(params)
    b, M = run.buf, plain["n_mixed"]
    flags = None
    for m in (M, 700):
        for delta in (scale * (0.25 + shift), 1e-3 + shift):
            print(f"[gpu-case] narrowed brackets {shift} {delta}: {m} cells", flush=True)
            cnt = torch.tensor([m, plain["n_band"]], dtype=torch.int32, device=run.dev)
            torch.cuda.synchronize()
            V.reconstruct_learned(run.ctx, run.mesh, run.alpha, b.mixed_idx, cnt, b.itf, mlp, delta)
            torch.cuda.synchronize()
            g = run.results()
            ok = plain["status"][:m] == V.CELL_OK
            st = g["status"][:m]
            assert np.isin(st[ok], [V.CELL_OK, V.CELL_LEARNED_FALLBACK]).all()
            np.testing.assert_allclose(g["alpha_got"][:m][ok], wl.alpha[g["mixed_idx"][:m]][ok], rtol=0, atol=1e-12)
            if m == M:
                flags = {} if flags is None else flags
                flags[delta] = st.copy()
            np.testing.assert_array_equal(st, flags[delta][:m])
    run.close()
    mlp.close()
