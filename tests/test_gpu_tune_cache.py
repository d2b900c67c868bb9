"""A line of the autotuner's cache counts only for the kernels it was timed with."""
import re

import pytest

from synth import workloads
from tests.test_gpu_teams import V  # noqa: F401  (a fixture)

pytestmark = pytest.mark.gpu


def test_lines_of_other_kernel_revisions_are_ignored(V, tmp_path):  # noqa: F811
    import torch
    from paper_2604_14938_amd import runner
    run = runner.PathRun(workloads.voronoi_bubble(n=12, seed=7, r=0.3), ctx=V.Context(0, stream=torch.cuda.Stream()))
    path = tmp_path / "tune.txt"

    def tune():
        return V.autotune(run.ctx, run.mesh, run.alpha, cache_path=str(path))

    assert not tune()[1]
    assert tune()[1]
    line = path.read_text().strip()
    rev = re.search(r" r(\d+) ", line)
    assert rev, line
    forced = line.rsplit(":", 1)[0] + ": 3 4 3 3"
    path.write_text(forced + "\n")
    assert tune()[1] and run.mesh.classes()["tune"][1] == 4
    for old in (" ", f" r{int(rev[1]) - 1} "):   # no revision, and the one before
        path.write_text(forced.replace(rev[0], old) + "\n")
        choice, hit = tune()
        assert not hit, path.read_text()
    run.close()
