"""The status and the evaluation count of a reconstruction that is given a
bracket per cell: with a fixed isovalue, where no search runs, and where an end
of the bracket is the isovalue itself.  One cell per group and in teams, against
the oracle."""
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


@pytest.mark.parametrize("kind", ["hex", "voronoi"])
def test_brackets_that_end_at_the_isovalue(V, kind):  # noqa: F811
    """Brackets from, to and about the isovalue of the plain search hold it
    (an end whose volume meets the tolerance is a result); brackets beside it
    do not, unless nothing of them lies in the cell's range."""
    import torch
    from paper_2604_14938_amd import runner
    wl, _ = _case(kind)
    om = oracle.OMesh(wl.mesh)
    geom = oracle.geometry(om)
    run = runner.PathRun(wl, ctx=V.Context(0, stream=torch.cuda.Stream()))
    run.step()
    full = run.results()
    b, M = run.buf, full["n_mixed"]
    feat = torch.empty(M, 32, dtype=torch.float32, device=run.dev)
    rng = torch.empty(M, 2, dtype=torch.float64, device=run.dev)
    V.features(run.ctx, run.mesh, run.alpha, b.mixed_idx, b.counts, feat, rng)
    torch.cuda.synchronize()
    W = rng[:, 1].cpu().numpy()
    opts = V.recon_opts(bracket=V.BRACKET_HINT)
    for m in COUNTS:
        m = m or M
        cnt = torch.tensor([m, full["n_band"]], dtype=torch.int32, device=run.dev)
        torch.cuda.synchronize()
        V.reconstruct(run.ctx, run.mesh, run.alpha, b.mixed_idx, cnt, b.itf)
        plain = _first(run.results(), m)
        s, w, idx, ok = plain["s"], 0.02 * W[:m], plain["mixed_idx"], plain["status"] == V.CELL_OK
        a = wl.alpha[idx]
        # where the search ended within the tolerance, not at adjacent doubles
        met = ok & (np.abs(plain["alpha_got"] - a) <= 1e-13 * np.minimum(a, 1.0 - a))
        assert met.mean() > 0.95
        for name, lo, hi in (("from", s, s + w), ("to", s - w, s), ("point", s, s), ("about", s - w, s + 0.7 * w),
                             ("above", s + 0.1 * w, s + w), ("below", s - w, s - 0.1 * w)):
            print(f"[gpu-case] brackets {kind} {name}: {m} of {M} cells", flush=True)
            l, h = (torch.as_tensor(x, dtype=torch.float64, device=run.dev) for x in (lo, hi))
            torch.cuda.synchronize()
            V.reconstruct(run.ctx, run.mesh, run.alpha, b.mixed_idx, cnt, b.itf, opts, l, h)
            g = _first(run.results(), m)
            if name in ("from", "to", "point"):
                want = np.full(m, V.CELL_OK)
            else:
                dl, dh = np.full(wl.mesh.n_cells, np.nan), np.full(wl.mesh.n_cells, np.nan)
                dl[idx], dh[idx] = lo, hi
                want = oracle.reconstruct(om, wl.alpha, geom, hint_lo=dl, hint_hi=dh, cells=idx)["status"][idx]
                assert ((want == V.CELL_LEARNED_FALLBACK).mean() > 0.5) == (name != "about")
            wrong = np.nonzero((met if name in ("from", "to", "point") else ok) & (g["status"] != want))[0]
            assert wrong.size == 0, (name, m, wrong.size, idx[wrong[:4]], g["status"][wrong[:4]], want[wrong[:4]])
            np.testing.assert_allclose(g["alpha_got"][ok], a[ok], rtol=0, atol=1e-12)
    run.close()


@pytest.mark.parametrize("kind,tune", [("hex", None), ("voronoi", None), ("voronoi", (12, 3, 26, 3))])
def test_the_network_predicts_the_same_bits(V, kind, tune):  # noqa: F811
    """The brackets of one, four and sixteen cells per wavefront against those
    of the wavefront kernel, bit for bit."""
    import torch
    from paper_2604_14938_amd import runner, train
    wl, _ = _case(kind)
    params, scale, _ = train.load()
    run = runner.PathRun(wl, ctx=V.Context(0, stream=torch.cuda.Stream()))
    mlp = V.Mlp(run.ctx)
    mlp.set_params(params)
    run.step()
    full = run.results()
    b, M = run.buf, full["n_mixed"]

    def brackets(m):
        lo, hi = (torch.zeros(M, dtype=torch.float64, device=run.dev) for _ in range(2))
        cnt = torch.tensor([m, full["n_band"]], dtype=torch.int32, device=run.dev)
        torch.cuda.synchronize()
        V.reconstruct_learned(run.ctx, run.mesh, run.alpha, b.mixed_idx, cnt, b.itf, mlp, scale, None, lo, hi)
        torch.cuda.synchronize()
        return lo[:m].cpu().numpy(), hi[:m].cpu().numpy()

    group = run.mesh.classes()["tune"] if tune is None else list(tune)
    run.mesh.set_tune([3, 3, 3, 3])
    ref = brackets(M)
    assert np.isfinite(ref[0]).mean() > 0.99
    run.mesh.set_tune(group)
    for m in (M, 5000, 3000, 900, 17, 1):
        print(f"[gpu-case] network bits {kind} {tune}: {m} of {M} cells", flush=True)
        for g, r in zip(brackets(m), ref):
            np.testing.assert_array_equal(g, r[:m])
    run.close()
    mlp.close()


@pytest.mark.parametrize("kind", ["hex", "voronoi"])
def test_the_network_beside_fractions_that_are_no_numbers(V, kind):  # noqa: F811
    """Cells next to a NaN fraction get no usable inputs and are searched as
    without the network; the others do not notice."""
    import dataclasses

    import torch
    from paper_2604_14938_amd import runner, train
    base, _ = _case(kind)
    alpha = base.alpha.copy()
    mixed = np.nonzero((alpha > 1e-8) & (alpha < 1 - 1e-8))[0]
    alpha[mixed[::101]] = np.nan
    wl = dataclasses.replace(base, alpha=alpha)
    params, scale, _ = train.load()
    run = runner.PathRun(wl, ctx=V.Context(0, stream=torch.cuda.Stream()))
    mlp = V.Mlp(run.ctx)
    mlp.set_params(params)
    run.step()
    full = run.results()
    b = run.buf
    for m in (full["n_mixed"], 900):
        print(f"[gpu-case] NaN fractions {kind}: {m} cells", flush=True)
        cnt = torch.tensor([m, full["n_band"]], dtype=torch.int32, device=run.dev)
        torch.cuda.synchronize()
        V.reconstruct(run.ctx, run.mesh, run.alpha, b.mixed_idx, cnt, b.itf)
        plain = _first(run.results(), m)["status"]
        V.reconstruct_learned(run.ctx, run.mesh, run.alpha, b.mixed_idx, cnt, b.itf, mlp, scale)
        st = _first(run.results(), m)["status"]
        st = np.where((st == V.CELL_LEARNED_FALLBACK) & (plain == V.CELL_OK), plain, st)
        np.testing.assert_array_equal(st, plain)
    run.close()
    mlp.close()
