"""The device-wide sort at its tiles' edges (2,048 keys, and 4,096 from 2^23),
over digits of 6 to 10 bits: the plan's order must be the stable order of the
queries' keys, which a plan of at most 8,192 queries (another sort) gives."""
import numpy as np
import pytest

import synth
from harness import Run, log

pytestmark = pytest.mark.gpu


def plan_arrays(r):
    n = r.nq
    a = (4 * n + 255) // 256 * 256
    p = r.plan.cpu().numpy()
    return (p[:4 * n].view(np.uint32).astype(np.int64), p[a:a + 4 * n].view(np.uint32).astype(np.int64))


@pytest.mark.parametrize("n,cells", [(8193, (9, 7, 8)), (10239, (3, 3, 3)), (10240, (6, 6, 6)), (10241, (40, 40, 40)),
                                     (20481, (60, 60, 60)), (8388607, (40, 40, 40)), (8388608, (60, 60, 60)),
                                     (8388609, (9, 7, 8)), (8392705, (40, 40, 40))])
def test_device_sort_at_tile_edges(n, cells):
    g = synth.random_gaussians(161, 8)
    base = synth.random_points(162, 9000, -0.05, 1.05)
    log(f"case {n} queries, cells {cells}")
    key = np.empty(9000, np.int64)
    for a in (0, 4500):
        small = Run(g, cells, "points", points=base[a:a + 4500])
        small.forward()
        k, o = plan_arrays(small)
        key[a + o] = k
    repeats = -(-n // 9000)  # equal keys far apart
    key = np.tile(key, repeats)[:n]
    r = Run(g, cells, "points", points=np.tile(base, (repeats, 1))[:n])
    r.forward()
    k, o = plan_arrays(r)
    want = np.argsort(key, kind="stable")
    np.testing.assert_array_equal(o, want)
    np.testing.assert_array_equal(k, key[want])
