"""The index of sets at the sizes where the preprocess changes the number of
Gaussians a wave takes (8, 16, 32, 64), with partly filled last waves and
with boxes of both row-run forms and of none in one wave, against the oracle."""
import numpy as np
import pytest

import synth
from harness import Run, check_index, log

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 7, 9, 65, 24576, 24577, 65535, 65537, 98304, 98305])
def test_index_at_the_wave_sizes(n):
    g = synth.random_gaussians(151, n, log_mu=np.log(0.45 * n ** (-1 / 3)), log_sd=0.8)
    log(f"case {n} Gaussians")
    c = max(3, int(0.9 * n ** (1 / 3)))
    check_index(Run(g, (c + 3, c, c + 1), "points", points=synth.random_points(152, 64)), reach_sample=500)
