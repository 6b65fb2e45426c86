"""The grid forward tests the cutoff on the same float32 Q as the other
forwards and the pair counts, whatever the voxels of a cell and however small
or flat the Gaussians are against it."""
import numpy as np
import pytest

import oracle
import synth
from harness import TAU, Run, check_forward, log

pytestmark = pytest.mark.gpu

CELLS = (9, 8, 7)
SHAPES = [(1, 1, 1), (2, 1, 1), (3, 1, 1), (2, 2, 1), (5, 1, 1), (2, 2, 2), (3, 3, 1), (4, 2, 2), (17, 1, 1), (4, 4, 2),
          (11, 3, 1), (3, 4, 4), (7, 3, 3)]


def unit_quaternions(rng, n):
    q = rng.standard_normal((n, 4))
    return q / np.linalg.norm(q, axis=1, keepdims=True)


def on_cutoff(rng, p, scale, q, spread):
    """Means that put the points p on the cutoff ellipsoids, within `spread`
    of their radius."""
    w, x, y, z = q.T
    R = np.stack([np.stack([1 - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y)], -1),
                  np.stack([2 * (x * y + w * z), 1 - 2 * (x * x + z * z), 2 * (y * z - w * x)], -1),
                  np.stack([2 * (x * z - w * y), 2 * (y * z + w * x), 1 - 2 * (x * x + y * y)], -1)], 1)
    d = rng.standard_normal(p.shape)
    d /= np.linalg.norm(d, axis=1, keepdims=True)
    d *= np.sqrt(2.0 * np.log(1.0 / TAU)) * (1.0 + rng.uniform(-spread, spread, (len(p), 1)))
    return p - np.einsum("nij,nj->ni", R, d * scale)


@pytest.mark.parametrize("per_cell", SHAPES)
def test_one_gaussian_a_cell_gives_the_voxel_lists_bits(per_cell):
    """Where a cell lists one Gaussian, the sums are w 2^-Q' and w v 2^-Q' in
    every forward, so grid and voxel list must agree bit for bit, and the
    grid's defined voxels are the pairs that sample_pair_counts says
    contribute (w = 4, so that G >= tau is above the threshold). Flat
    Gaussians (30 to 1) sixty times smaller than the cells' diagonal, each
    with one voxel centre at its cutoff."""
    import paper_2607_01164_amd as gs
    rng = np.random.default_rng(181)
    dims = tuple(c * r for c, r in zip(CELLS, per_cell))
    n = CELLS[0] * CELLS[1] * CELLS[2]
    cell = np.stack([np.arange(n) % CELLS[0], np.arange(n) // CELLS[0] % CELLS[1], np.arange(n) // (CELLS[0] * CELLS[1])], 1)
    # the voxel nearest to the cell's middle: its Gaussian's box stays inside the cell
    p = (cell * np.asarray(per_cell) + (np.asarray(per_cell) - 1) // 2 + 0.5) / np.asarray(dims)
    size = np.sqrt(sum(1.0 / c ** 2 for c in CELLS)) / 60.0
    scale = size * np.stack([np.ones(n), rng.uniform(0.3, 1.0, n), np.full(n, 1.0 / 30.0)], 1)
    q = unit_quaternions(rng, n)
    f = np.float32
    g = synth.Gaussians(on_cutoff(rng, p, scale, q, 1e-5).astype(f), scale.astype(f), q.astype(f),
                        rng.uniform(0.1, 1.0, n).astype(f), np.full(n, 4.0, f))
    log(f"case one Gaussian a cell, cells of {per_cell} voxels")
    r = Run(g, CELLS, "grid", dims=dims)
    per = np.diff(r.index_arrays()[2].astype(np.int64))
    one = per <= 1
    assert one.mean() > 0.7
    phi, inf = r.forward()
    v = Run(g, CELLS, "voxels", dims=dims, ids=np.arange(r.nq, dtype=np.uint32))
    pv, iv = v.forward()
    x = np.arange(r.nq)
    vox = np.stack([x % dims[0], x // dims[0] % dims[1], x // (dims[0] * dims[1])], 1) // np.asarray(per_cell)
    sel = one[vox[:, 0] + CELLS[0] * (vox[:, 1] + CELLS[1] * vox[:, 2])]
    np.testing.assert_array_equal(phi[sel].view(np.uint32), pv[sel].view(np.uint32))
    np.testing.assert_array_equal(inf[sel].view(np.uint32), iv[sel].view(np.uint32))
    work = gs.alloc_backward_work(r.index, r.query, "cuda")
    _, hits = gs.sample_pair_counts(r.index, r.query, None, work)
    log(f"  {hits} contributing, {int((inf > 0).sum())} defined, one Gaussian in {one.mean():.2f} of the cells")
    if one.all():
        assert hits == int((inf > 0).sum())


@pytest.mark.parametrize("per_cell", SHAPES + [(5, 13, 1)])
def test_flat_gaussians_at_their_cutoff(per_cell):
    """Lists of a few dozen flat Gaussians from the cells' size down to a
    sixtieth of it, under a few wide ones: every output against the oracle,
    whose bar lets a pair change sides only within float32 rounding of U (p -
    mu)."""
    rng = np.random.default_rng(182)
    dims = tuple(c * r for c, r in zip(CELLS, per_cell))
    n = 12000
    vox = np.stack([rng.integers(0, d, n) for d in dims], 1)
    p = oracle.voxel_centers(dims, (0, 0, 0), (1, 1, 1),
                             ids=(vox[:, 0] + dims[0] * (vox[:, 1] + dims[1] * vox[:, 2])).astype(np.uint32))
    size = np.sqrt(sum(1.0 / c ** 2 for c in CELLS)) / np.exp(rng.uniform(np.log(3.0), np.log(60.0), n))
    scale = size[:, None] * np.stack([np.ones(n), rng.uniform(0.1, 1.0, n), np.full(n, 1.0 / 30.0)], 1)
    q = unit_quaternions(rng, n)
    mean = on_cutoff(rng, p, scale, q, 1e-4)
    wide = 6
    f = np.float32
    g = synth.Gaussians(np.concatenate([mean, rng.uniform(0.2, 0.8, (wide, 3))]).astype(f),
                        np.concatenate([scale, np.full((wide, 3), 0.4)]).astype(f),
                        np.concatenate([q, np.tile([1.0, 0, 0, 0], (wide, 1))]).astype(f),
                        rng.random(n + wide).astype(f), np.concatenate([rng.uniform(0.5, 1.0, n), np.ones(wide)]).astype(f))
    log(f"case flat Gaussians, cells of {per_cell} voxels")
    r = Run(g, CELLS, "grid", dims=dims)
    phi, inf = r.forward()
    check_forward(r, phi, inf, label=f"flat {per_cell}")
