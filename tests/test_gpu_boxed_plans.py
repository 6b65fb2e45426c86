"""Plans of boxed launches (320 queries a cell or more on average), whose
order is refined by place and whose positions carry the places: every way of
filling and using them, for points, voxel lists and jitter, with gs_sample's
outputs as the reference, bit for bit."""
import numpy as np
import pytest

import synth
from harness import Run, check_forward, log

pytestmark = pytest.mark.gpu

CELLS = (3, 2, 2)  # 12 cells
DIMS = (42, 40, 38)


def boxed_run(kind, n):
    """n queries, some of them outside the domain."""
    g = synth.random_gaussians(171, 1200, log_mu=np.log(0.05), log_sd=0.6)
    if kind == "points":
        return Run(g, CELLS, kind, points=synth.random_points(172, n, -0.01, 1.01))
    nvox = DIMS[0] * DIMS[1] * DIMS[2]
    ids = np.random.default_rng(173).choice(nvox, size=n, replace=False).astype(np.uint32)
    ids[:5] = [nvox, nvox + 1, 0xFFFFFFFF, nvox * 2, nvox + 7]
    u = synth.jitter_offsets(174, n) if kind == "jitter" else None
    return Run(g, CELLS, kind, dims=DIMS, ids=ids, offsets=u)


def planned(r):
    import torch
    v, i = torch.empty_like(r.value), torch.empty_like(r.influence)
    r.gs.gs_sample_planned(r.dg, r.index, r.query, v, i, r.plan)
    torch.cuda.synchronize()
    return v.cpu().numpy(), i.cpu().numpy()


def places(r):
    """keys, refined order and positions (with the places in w) of the plan."""
    n = r.nq
    a = (4 * n + 255) // 256 * 256
    p = r.plan.cpu().numpy()
    at = p.tobytes()
    end = len(at) - ((8 * n + 255) // 256 * 256) - ((16 * (n + 64) + 255) // 256 * 256)
    return p[:4 * n], p[3 * a:3 * a + 4 * n], p[end:end + 16 * n]


@pytest.mark.parametrize("n", [6000, 30000])  # 500 and 2,500 a cell: both box sizes
@pytest.mark.parametrize("kind", ["points", "voxels", "jitter"])
def test_a_plan_serves_every_forward(kind, n):
    log(f"case boxed plans, {n} {kind}")
    r = boxed_run(kind, n)
    assert r.nq >= 320 * 12
    phi, inf = r.forward()
    sel = np.arange(5, n) if kind != "points" else None
    check_forward(r, phi, inf, sel=sel, label=f"boxed {kind}")
    want = places(r)
    assert len(np.unique(want[2].view(np.uint32).reshape(-1, 4)[:, 3])) > 8, "the places are in w"

    r.plan.zero_()
    r.gs.gs_plan_queries(r.query, r.grid, r.plan)
    for after in ("gs_plan_queries", "gs_sample_planned", "gs_sample_gaussian_major"):
        if after == "gs_sample_gaussian_major":
            r.forward_gm()
            sel = np.arange(5, n) if kind != "points" else None
            check_forward(r, r.phi_np, r.inf_np, sel=sel, label="gaussian-major")
        if after != "gs_plan_queries":  # (that fills a plan for a forward, which writes the rest)
            for a, b in zip(want, places(r)):
                np.testing.assert_array_equal(a, b, err_msg=f"the plan after {after}")
        v, i = planned(r)
        np.testing.assert_array_equal(v.view(np.uint32), phi.view(np.uint32), err_msg=f"after {after}")
        np.testing.assert_array_equal(i.view(np.uint32), inf.view(np.uint32), err_msg=f"after {after}")
