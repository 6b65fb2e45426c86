"""The grid backward's rows of voxels: cut to the cutoff ellipsoid in y and z
and along x, handed to lanes by marks. Every gradient against the oracle, for
Gaussians from far below a voxel to wider than the grid, cut by the box on
every side, and for both numbers of Gaussians a wave."""
import numpy as np
import pytest

import oracle
import synth
from harness import Run, check_backward, check_forward, log, masked_cotangents

pytestmark = pytest.mark.gpu


def mixed_gaussians(seed, n):
    """Scales from 0.002 to 0.6 per axis, means inside and around the box."""
    rng = np.random.default_rng(seed)
    g = synth.random_gaussians(seed, n, log_mu=np.log(0.03), log_sd=0.4)
    wide = rng.random(n) < 0.1
    s = np.where(wide[:, None], np.exp(rng.uniform(np.log(0.002), np.log(0.6), (n, 3))), g.scale)
    mean = rng.uniform(-0.1, 1.1, (n, 3))
    f = np.float32
    return synth.Gaussians(mean.astype(f), s.astype(f), g.rot, g.value, g.weight)


@pytest.mark.parametrize("dims,cells", [((16, 16, 16), (8, 8, 8)), ((33, 20, 7), (11, 5, 7)), ((64, 1, 5), (2, 1, 5)),
                                        ((130, 6, 6), (1, 1, 1))])
def test_grid_gradients(dims, cells):
    g = mixed_gaussians(131, 400)
    log(f"case grid gradients {dims}, cells {cells}")
    r = Run(g, cells, "grid", dims=dims, lo=(0.1, -0.2, 0.0), hi=(1.0, 1.0, 0.9))
    phi, inf = r.forward()
    ref, _ = check_forward(r, phi, inf, label="grid")
    gv, gi = synth.random_normal(132, r.nq), synth.random_normal(133, r.nq)
    gv, gi, _ = masked_cotangents(ref, gv, gi)
    check_backward(r, r.backward(gv, gi), np.arange(g.n), np.arange(r.nq), gv, gi, label="grid")


def test_grid_gradients_four_gaussians_a_wave():
    """66,001 Gaussians (four a wave), and the pair count against the pairs
    that contribute: rows cut to the cutoff test few others."""
    import paper_2607_01164_amd as gs
    g = synth.random_gaussians(134, 66001, log_mu=np.log(0.012), log_sd=0.4)
    log("case grid gradients, four a wave")
    r = Run(g, (20, 20, 20), "grid", dims=(40, 40, 40))
    phi, inf = r.forward()
    ref = oracle.forward(g, r.positions())
    gv, gi = synth.random_normal(135, r.nq), synth.random_normal(136, r.nq)
    gv, gi, _ = masked_cotangents(ref, gv, gi)
    sel = np.random.default_rng(137).choice(g.n, 2000, replace=False)
    check_backward(r, r.backward(gv, gi), sel, np.arange(r.nq), gv, gi, label="four a wave")
    work = gs.alloc_backward_work(r.index, r.query, "cuda")
    tests = gs.backward_pair_count(r.index, r.query, None, work)
    hits = int(ref.ncontrib.sum())
    log(f"  {tests} tests, {hits} contributing")
    assert hits <= tests <= 1.1 * hits
