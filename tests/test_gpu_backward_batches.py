"""The backward's batches of 64 rows where several Gaussians share a wave
(65,536 Gaussians or more): a last batch of one to three rows holds rows of
a Gaussian that a lane past those rows describes."""
import numpy as np
import pytest

import synth
from harness import Run, log

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["points", "grid"])
@pytest.mark.parametrize("scale", [0.0095, 0.011])
def test_every_pair_counts_in_last_batches_of_few_rows(kind, scale):
    """With unit cotangents the gradients add up to what the forward summed:
    sum dL/dv = number of defined queries (dL/dPhi = 1, dL/dI = 0) and
    sum w dL/dw = sum I (dL/dPhi = 0, dL/dI = 1). Every term is positive, so
    a lost pair shows. Four Gaussians of some 9 to 16 rows share a wave: among
    70,001 / 4 waves some hundreds end in a batch of one to three rows. Bar:
    each gradient sums at most 512 pairs in float32, (512 / 64 + 24) 2^-24 =
    1.9e-6 of its sum, and each I as many, 512 2^-24 = 3.1e-5 at worst and
    their square root typically; 1e-5 of the total."""
    n = 70001
    g = synth.random_gaussians(91, n, log_mu=np.log(scale), log_sd=0.25)
    log(f"case last batches, {kind}, scale {scale}")
    if kind == "points":
        r = Run(g, (33, 35, 31), "points", points=synth.random_points(92, 40000))
    else:
        r = Run(g, (33, 35, 31), "grid", dims=(33, 35, 31))
    assert r.index.n_pairs < 32 * n  # four Gaussians a wave
    r.forward()
    inf = r.inf_np.astype(np.float64)
    one, zero = np.ones(r.nq, np.float32), np.zeros(r.nq, np.float32)
    dv = r.backward(one, zero)[:, 10].astype(np.float64).sum()
    dw = (r.backward(zero, one)[:, 11].astype(np.float64) * g.weight).sum()
    log(f"  dv {dv / (inf > 0).sum() - 1:.2e} dw {dw / inf.sum() - 1:.2e}")
    assert dv == pytest.approx((inf > 0).sum(), rel=1e-5)
    assert dw == pytest.approx(inf.sum(), rel=1e-5)
