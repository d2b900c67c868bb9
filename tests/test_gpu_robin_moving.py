"""The interface coupling on one mesh as its interface moves, shrinks and goes:
each call gives what a mesh that never saw another interface gives."""
import dataclasses

import numpy as np
import pytest

from synth import meshes, workloads
from tests.test_gpu_robin import K_L, K_V, R, _fwd, _gpu, _say  # noqa: F401  (R is a fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["hex", "voronoi"])
def test_moving_interface(R, kind):  # noqa: F811
    import torch
    from paper_2604_14938_amd import vofpc as V
    mesh = meshes.hex_mesh(24) if kind == "hex" else meshes.voronoi_box_mesh(12, seed=3)
    wls = [workloads.random_bubbles(mesh, seed=s, n_max=n, K=12, r_hi_h=3.0) for s, n in ((1, 12), (2, 3), (3, 12))]
    wls.insert(2, dataclasses.replace(wls[0], alpha=np.ones_like(wls[0].alpha)))   # no interface at all
    _say(f"coupling of a moving interface, {kind}: {[w.n_mixed for w in wls]} mixed")
    _, run, out = _gpu(R, wls[0])
    b = run.buf
    for wl in wls[1:] + wls[:1]:
        run.alpha.copy_(torch.as_tensor(wl.alpha))
        run.T.copy_(torch.as_tensor(wl.T))
        run.Tb.copy_(torch.as_tensor(wl.T_bface))
        torch.cuda.synchronize()
        run.step()
        torch.cuda.synchronize()
        V.robin(run.ctx, run.mesh, run.alpha, b.mixed_idx, b.band_idx, b.counts, b.itf, K_L, K_V, **_fwd(out))
        torch.cuda.synchronize()
        want, fresh, _ = _gpu(R, wl)
        n, nb = int(out["n_face"][0]), len(want["band_idx"])
        assert n == want["n_face"]
        np.testing.assert_array_equal(out["a_diag"][:nb].cpu().numpy(), want["a_diag"])
        order, order_w = (np.argsort(f[:n]) for f in (out["face_idx"].cpu().numpy(), want["face_idx"]))
        for k in ("face_idx", "face_area"):
            np.testing.assert_array_equal(out[k][:n].cpu().numpy()[order], want[k][:n][order_w])
        np.testing.assert_array_equal(out["face_a"].cpu().numpy()[:, :n][:, order], want["face_a"][:, :n][:, order_w])
        fresh.close()
    run.close()
