"""Which classes' cells the bench counts for a class kernel's time."""
import numpy as np
import pytest

import bench


@pytest.mark.parametrize("cells,ms,kc,want", [
    ([2097287, 5011108, 17892, 0], [0.30, 1.28, -1.0, -1.0], 1, [1, 2]),      # class 2 rides with class 1
    ([12, 1443, 3, 0], [-1.0, 0.05, -1.0, -1.0], 1, [0, 1, 2]),               # both neighbours ride
    ([2097287, 5011108, 17892, 0], [0.35, 1.10, 0.07, -1.0], 1, [1]),         # a kernel each
    ([2097287, 5011108, 17892, 0], [1.50, 1.28, -1.0, -1.0], 0, [0]),
])
def test_riding_classes_count_with_the_usual_one(cells, ms, kc, want):
    cls = {"cells": cells, "bucketed": True}
    assert int(np.argmax(ms)) == kc
    assert bench.kernel_classes(cls, np.array(ms), kc) == want
