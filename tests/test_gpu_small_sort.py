"""Orderings of at most 8,192 queries or Gaussians, sorted by one workgroup:
the plan's keys, order and ranges against those of a larger batch (the
device-wide sort) that holds the same queries, and gradients, which every
Gaussian's place in the visiting order enters."""
import numpy as np
import pytest

import synth
from harness import Run, check_backward, check_forward, log, masked_cotangents

pytestmark = pytest.mark.gpu

CELLS = (9, 7, 8)
NC = 9 * 7 * 8


def plan_arrays(r):
    n = r.nq
    a = (4 * n + 255) // 256 * 256
    p = r.plan.cpu().numpy()
    keys = p[:4 * n].view(np.uint32).astype(np.int64)
    order = p[a:a + 4 * n].view(np.uint32).astype(np.int64)
    poff = p[4 * a:4 * a + 4 * (4 * NC + 2)].view(np.uint32).astype(np.int64)
    return keys, order, poff


@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 1000, 1024, 1025, 4097, 8191, 8192])
def test_small_query_order(n):
    g = synth.random_gaussians(141, 50)
    pts = synth.random_points(142, 9000, -0.1, 1.1)
    pts[5:40] = pts[5]  # equal keys keep their order
    log(f"case small order of {n}")
    big, small = Run(g, CELLS, "points", points=pts), Run(g, CELLS, "points", points=pts[:n])
    big.forward()
    small.forward()
    bk, bo, _ = plan_arrays(big)
    key = np.empty(9000, np.int64)
    key[bo] = bk
    k, o, off = plan_arrays(small)
    want = np.argsort(key[:n], kind="stable")
    np.testing.assert_array_equal(o, want)
    np.testing.assert_array_equal(k, key[:n][want])
    np.testing.assert_array_equal(off, np.searchsorted(k, np.arange(4 * NC + 2), side="left"))


@pytest.mark.parametrize("n", [1, 65, 1025, 8192])
def test_gradients_with_a_small_gaussian_order(n):
    g = synth.random_gaussians(143, n, log_mu=np.log(0.4 * n ** (-1 / 3)), log_sd=0.5)
    log(f"case {n} Gaussians")
    r = Run(g, CELLS, "points", points=synth.random_points(144, 3000))
    phi, inf = r.forward()
    ref, _ = check_forward(r, phi, inf, label="small order")
    gv, gi = synth.random_normal(145, r.nq), synth.random_normal(146, r.nq)
    gv, gi, _ = masked_cotangents(ref, gv, gi)
    check_backward(r, r.backward(gv, gi), np.arange(g.n), np.arange(r.nq), gv, gi, label="small order")
