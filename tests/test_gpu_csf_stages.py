"""The stages of the curvature chain at the edges of their launches: eight and
sixteen lanes a cell, one turn and several turns of a wavefront, cell counts
that end inside a wavefront, cells with more faces than lanes, and rings that
reach the boundary."""
import numpy as np
import pytest

from synth import fields, meshes
from tests import test_gpu_csf as base
from tests.test_gpu_csf import V  # noqa: F401  (a fixture)

pytestmark = pytest.mark.gpu

MESHES = {"hex_odd": lambda: meshes.hex_mesh(13), "hex_turns": lambda: meshes.hex_mesh(75),
          "vor": lambda: meshes.voronoi_box_mesh(9, seed=4, jitter=0.45)}


@pytest.mark.parametrize("name,n_smooth,with_force", [("hex_odd", 1, False), ("hex_odd", 3, True),
                                                      ("hex_turns", 2, True), ("vor", 1, True), ("vor", 2, False)])
def test_stages(V, monkeypatch, name, n_smooth, with_force):  # noqa: F811
    def case(_):
        m = MESHES[name]()
        centre, r = ([0.2, 0.24, 0.22], 0.13) if name != "hex_turns" else ([0.41, 0.5, 0.53], 0.35)
        return m, 1.0 - fields.sphere_alpha(m, np.array([[*centre, r]]), K=12)
    m = case(None)[0]
    if name == "vor":
        assert np.diff(m.cell_face_off).max() > 16
    if name == "hex_turns":
        assert m.n_cells > 48 * 256 * 4 * 8
    monkeypatch.setattr(base, "_case", case)
    base.test_curvature_matches_oracle(V, name, n_smooth, with_force)
