"""Boxed launches (2^21 queries and 320 a cell or more that meet long lists),
whose plans are refined by place and whose positions carry the places: every
way of filling and using the plan, for points, voxel lists and jitter, with
gs_sample's outputs as the reference, bit for bit; their exactness; coarse
cells; and more queries than a launch has threads."""
import numpy as np
import pytest

import synth
from harness import TAU, Run, check_forward, is_boxed, log, with_long_lists

pytestmark = pytest.mark.gpu

DIMS = (140, 130, 132)
N = (1 << 21) + 5003


def plan_run(kind, cells, lists):
    """N queries, some of them outside the domain, on lists of `lists` pairs and
    more."""
    g = with_long_lists(synth.random_gaussians(171, 1200, log_mu=np.log(0.03), log_sd=0.6), lists)
    if kind == "points":
        return Run(g, cells, kind, points=synth.random_points(172, N, -0.01, 1.01))
    nvox = DIMS[0] * DIMS[1] * DIMS[2]
    ids = np.random.default_rng(173).choice(nvox, size=N, replace=False).astype(np.uint32)
    ids[:5] = [nvox, nvox + 1, 0xFFFFFFFF, nvox * 2, nvox + 7]
    u = synth.jitter_offsets(174, N) if kind == "jitter" else None
    return Run(g, cells, kind, dims=DIMS, ids=ids, offsets=u)


def planned(r):
    import torch
    v, i = torch.empty_like(r.value), torch.empty_like(r.influence)
    r.gs.gs_sample_planned(r.dg, r.index, r.query, v, i, r.plan)
    torch.cuda.synchronize()
    return v.cpu().numpy(), i.cpu().numpy()


def plan_parts(r):
    """keys, order and positions (with the places in w) of the plan."""
    n = r.nq
    a = (4 * n + 255) // 256 * 256
    p = r.plan.cpu().numpy()
    at = len(p) - ((8 * n + 255) // 256 * 256) - ((16 * (n + 64) + 255) // 256 * 256)
    return p[:4 * n], p[a:a + 4 * n], p[at:at + 16 * n]


@pytest.mark.parametrize("cells", [(17, 16, 15), (3, 2, 2)])  # 515 and 175,179 a cell: both box sizes
@pytest.mark.parametrize("kind,lists", [("points", 340), ("voxels", 340), ("jitter", 340), ("points", 70)])
def test_a_plan_serves_every_forward(kind, lists, cells):
    """(Lists of 70: asked, and found not to be boxed.)"""
    log(f"case plans, {kind}, cells {cells}, lists of {lists}")
    r = plan_run(kind, cells, lists)
    phi, inf = r.forward()
    assert is_boxed(r) == (lists >= 320) and r.index.n_pairs >= 60 * np.prod(cells)
    sel = np.sort(np.random.default_rng(178).choice(np.arange(5, N), 20000, replace=False))
    check_forward(r, phi, inf, sel=sel, label=f"boxed {kind}")
    want = plan_parts(r)
    places = np.unique(want[2].view(np.uint32).reshape(-1, 4)[:, 3])
    assert (len(places) > 3) == is_boxed(r), "the places are in w"

    r.plan.zero_()
    r.gs.gs_plan_queries(r.query, r.grid, r.plan)
    for after in ("gs_plan_queries", "gs_sample_planned", "gs_sample_gaussian_major"):
        if after == "gs_sample_gaussian_major":
            r.forward_gm()
            check_forward(r, r.phi_np, r.inf_np, sel=sel, label="gaussian-major")
        if after != "gs_plan_queries":  # (that fills a plan for a forward, which writes the rest)
            for a, b in zip(want, plan_parts(r)):
                np.testing.assert_array_equal(a, b, err_msg=f"the plan after {after}")
        v, i = planned(r)
        np.testing.assert_array_equal(v.view(np.uint32), phi.view(np.uint32), err_msg=f"after {after}")
        np.testing.assert_array_equal(i.view(np.uint32), inf.view(np.uint32), err_msg=f"after {after}")


@pytest.mark.parametrize("kind", ["points", "voxels"])
def test_a_plan_serves_another_index(kind):
    """A plan that a boxed forward has reordered, sampled with an index whose
    launches are not boxed, and with the first one again."""
    cells = (17, 16, 15)
    log(f"case plans, another index, {kind}")
    r, other = plan_run(kind, cells, 340), plan_run(kind, cells, 70)
    phi, inf = r.forward()
    other.forward()
    assert is_boxed(r) and not is_boxed(other)
    other.plan = r.plan
    v, i = planned(other)
    sel = np.sort(np.random.default_rng(179).choice(np.arange(5, N), 20000, replace=False))
    check_forward(other, v, i, sel=sel, label=f"another index, {kind}")
    v, i = planned(r)
    np.testing.assert_array_equal(v.view(np.uint32), phi.view(np.uint32))
    np.testing.assert_array_equal(i.view(np.uint32), inf.view(np.uint32))


@pytest.mark.parametrize("cells", [(13, 12, 11), (8, 8, 8)])
def test_boxed_coarse_cells_keep_small_gaussians_exact(cells):
    """Cells that list a Gaussian far smaller than they are keep U (p - mu) in
    boxed launches too: tiny Gaussians with 300 or more points each on their
    cutoff surfaces, under wide ones that make every point defined. Every
    output within the oracle's bar."""
    rng = np.random.default_rng(179)
    nt, per = 3400, 620
    mean = rng.uniform(0.1, 0.9, (nt, 3))
    scale = 0.0003 * rng.uniform(1.0, 2.0, (nt, 3))
    q = rng.standard_normal((nt, 4))
    d = rng.standard_normal((nt, per, 3))
    d *= np.sqrt(2.0 * np.log(1.0 / TAU)) * (1.0 + rng.uniform(-1e-4, 1e-4, (nt, per, 1))) / \
        np.linalg.norm(d, axis=2, keepdims=True)
    pts = (mean[:, None] + np.einsum("nij,npj->npi", rotations(q), d * scale[:, None])).reshape(-1, 3)
    f = np.float32
    nw = 8
    g = synth.Gaussians(np.concatenate([mean, rng.uniform(0.2, 0.8, (nw, 3))]).astype(f),
                        np.concatenate([scale, np.full((nw, 3), 0.4)]).astype(f),
                        np.concatenate([q, np.tile([1.0, 0, 0, 0], (nw, 1))]).astype(f), rng.random(nt + nw).astype(f),
                        np.concatenate([rng.uniform(0.5, 1.0, nt), np.ones(nw)]).astype(f))
    log(f"case boxed coarse cells {cells}")
    r = Run(with_long_lists(g), cells, "points", points=pts)
    phi, inf = r.forward()
    assert is_boxed(r)
    sel = np.sort(rng.choice(len(pts), 200000, replace=False))
    _, stats = check_forward(r, phi, inf, sel=sel, label="boxed coarse cells")
    assert stats["defined"] > 0.9 * len(sel)


def rotations(q):
    q = q.astype(np.float64)
    w, x, y, z = (q / np.linalg.norm(q, axis=1, keepdims=True)).T
    return np.stack([np.stack([1 - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y)], -1),
                     np.stack([2 * (x * y + w * z), 1 - 2 * (x * x + z * z), 2 * (y * z - w * x)], -1),
                     np.stack([2 * (x * z - w * y), 2 * (y * z + w * x), 1 - 2 * (x * x + y * y)], -1)], 1)


@pytest.mark.parametrize("flat", [1, 5, 30])
@pytest.mark.parametrize("ratio", [6, 20, 60])
def test_boxed_sums_are_as_exact_as_the_unboxed_ones(flat, ratio):
    """The matrix products' Q' has the bits of the vector form's, which a launch
    of half the queries takes in the same cells, and errs no more. One
    Gaussian of some weight in every third cell (`flat` its axis ratio,
    `ratio` the cell's diagonal over its largest scale), so that I = w G and
    -log2(I / w) is Q'; the wide ones that lengthen the lists vanish in the
    sums. Bar: the rms error of Q' against 64 bits at most 1.03
    times the other launch's (150,000 pairs or more a side: sampling moves an
    rms by under 1 %)."""
    f = np.float32
    c, n, per = 12, 64, 33000
    rng = np.random.default_rng(175)
    k = np.arange(n)
    cell = np.stack([k % 4 * 3 + 1, k // 4 % 4 * 3 + 1, k // 16 * 3 + 1], 1)
    scale = (np.sqrt(3) / c / ratio * np.array([1.0, 1.0, 1.0 / flat]) * np.ones((n, 1))).astype(f)
    mean = ((cell + rng.uniform(0.1, 0.9, (n, 3))) / c).astype(f)
    q = rng.standard_normal((n, 4)).astype(f)
    R = rotations(q)
    d = rng.standard_normal((n, per, 3))
    d *= 3.03 * rng.uniform(0.7, 0.995, (n, per, 1)) / np.linalg.norm(d, axis=2, keepdims=True)
    pts = (mean[:, None] + np.einsum("nij,npj->npi", R, d * scale[:, None])).astype(f)
    x = pts.astype(np.float64) - mean[:, None].astype(np.float64)
    u = np.einsum("nij,npi->npj", R, x) / scale[:, None].astype(np.float64)
    Q = (u * u).sum(2) / 2 * np.log2(np.e)
    m = 340
    g = with_long_lists(synth.Gaussians(mean, scale, q, np.full(n, 0.5, f), np.full(n, 4.0, f)), m)

    def rms(queries):
        p, exact = pts[:, :queries], Q[:, :queries]
        r = Run(g, (c, c, c), "points", points=p.reshape(-1, 3))
        _, inf = r.forward()
        per_cell = np.diff(r.index_arrays()[2].astype(np.int64))
        t = p.astype(np.float64) * c
        at = np.clip(np.floor(t), 0, c - 1).astype(np.int64)
        # (float32 places a point within 1e-5 of a face in either cell)
        inside = (np.abs(t - np.round(t)) > 1e-5).all(2)
        key = at[..., 0] + c * (at[..., 1] + c * at[..., 2])
        held = np.bincount(key.ravel(), minlength=c ** 3)
        inf = inf.reshape(n, queries).astype(np.float64)
        # dense cells that the pair's Gaussian alone reaches, and not the next one
        ok = inside & (held[key] >= 64) & (per_cell[key] <= m + 1) & (inf > 0.01)
        e = -np.log2(inf[ok] / 4.0) - exact[ok]
        return r, np.sqrt((e * e).mean()), ok, inf.astype(np.float32)

    log(f"case exactness of boxed sums, axis ratio {flat}, cell / scale {ratio}")
    rb, boxed, okb, ib = rms(per)
    ru, plain, oku, iu = rms(per // 2)
    assert is_boxed(rb) and not is_boxed(ru)
    log(f"  rms error of Q': boxed {boxed:.3e} ({okb.sum()} pairs), unboxed {plain:.3e} ({oku.sum()})")
    both = okb[:, :per // 2] & oku
    assert both.sum() > 150000 and boxed <= 1.03 * plain
    np.testing.assert_array_equal(ib[:, :per // 2][both].view(np.uint32), iu[both].view(np.uint32))


def test_boxed_launch_of_more_than_2_30_queries():
    """A launch takes fewer than 2^32 threads, and the boxed walk gives 256 to
    every 64 queries: 2^30 + 2^21 queries, 2^21 points over and over, give
    the 2^21 points' bits over and over (their cells hold 32,768, the level of
    the larger counts too). About 70 GB of device memory."""
    import torch
    import paper_2607_01164_amd as gs
    from harness import dev_gauss
    if torch.cuda.get_device_properties(0).total_memory < 100 << 30:
        pytest.skip("needs 100 GB")
    log("case 2^30 + 2^21 queries")
    g = with_long_lists(synth.random_gaussians(176, 250, log_mu=np.log(0.1), log_sd=0.3), 650)
    base = torch.from_numpy(synth.random_points(177, 1 << 21)).cuda()
    dg, grid = dev_gauss(g), gs.make_grid((4, 4, 4))
    index = gs.build_index(dg, grid, 0.01)
    assert index.n_pairs >= 650 * 64  # a uniform launch's queries test as many: boxed both ways
    out = []
    for repeats in (1, (1 << 9) + 1):
        pts = base.repeat(repeats, 1)
        query = gs.Query.pts(pts)
        v = torch.empty(len(pts), dtype=torch.float32, device="cuda")
        i = torch.empty_like(v)
        plan = gs.alloc_plan(query, grid, "cuda")
        gs.gs_sample(dg, index, query, v, i, plan)
        torch.cuda.synchronize()
        out.append((v.view(repeats, -1), i.view(repeats, -1)))
        del pts, query, plan
    assert bool((out[0][1] > 0).any())
    for a, b in zip(*out):
        assert bool((b.view(torch.int32) == a.view(torch.int32)).all())
    del out, base, index
    torch.cuda.empty_cache()
