"""The compaction of polyhedral meshes on both sides of the size at which the
band test moves from the cell pass to the face pass, with alphas at 1/2, NaN and
infinite: the lists against their definitions, two calls on one scratch."""
import numpy as np
import pytest

from synth import meshes
from tests.test_gpu_compact import EPS, V, _field, _say  # noqa: F401  (V is a fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [3, 11, 50, 51])
def test_polyhedral_lists(V, n):  # noqa: F811
    import torch
    m = meshes.voronoi_box_mesh(n, seed=9)
    N = m.n_cells
    assert (N < 262144) == (n < 51)
    a = _field(N, 5) if N > 1000 else np.random.default_rng(5).choice([0.0, 0.3, 0.7, 1.0], N)
    rng = np.random.default_rng(6)
    a[rng.choice(N, 20, replace=False)] = rng.choice([0.5, np.nan, np.inf, -np.inf, np.nextafter(0.5, 1)], 20)
    _say(f"compaction of {N} Voronoi cells")
    ctx = V.Context(0, stream=torch.cuda.Stream())
    mesh = V.Mesh(ctx, m)
    alpha = torch.as_tensor(a, device="cuda")
    mixed, band = (torch.full((N,), -7, dtype=torch.int32, device="cuda") for _ in range(2))
    counts = torch.full((2,), -7, dtype=torch.int32, device="cuda")
    want_m = np.nonzero((a > EPS) & (a < 1 - EPS))[0]
    in_band = (a > EPS) & (a < 1 - EPS)
    inner = m.face_neigh >= 0
    o, q = m.face_owner[inner], m.face_neigh[inner]
    cross = ((a[o] > 0.5) & (a[q] < 0.5)) | ((a[o] < 0.5) & (a[q] > 0.5))
    in_band[o[cross]] = True
    in_band[q[cross]] = True
    want_b = np.nonzero(in_band)[0]
    torch.cuda.synchronize()
    for _ in range(2):
        mixed.fill_(-7)
        torch.cuda.synchronize()
        V.compact(ctx, mesh, alpha, mixed, band, counts, eps_mixed=EPS)
        torch.cuda.synchronize()
        nm, nb = (int(x) for x in counts.cpu())
        assert (nm, nb) == (len(want_m), len(want_b))
        np.testing.assert_array_equal(mixed[:nm].cpu().numpy(), want_m)
        np.testing.assert_array_equal(band[:nb].cpu().numpy(), want_b)
        assert (mixed[nm:] == -7).all()
    mesh.close()
    ctx.close()
