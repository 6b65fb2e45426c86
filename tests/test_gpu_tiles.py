"""The forward's matrix tiles (16 queries x 16 candidates) at their edges, in
boxed launches (2^21 queries, 320 a cell and 320 pairs a query or more), whose
dense cells are cut into boxes by their query count; and grid cells whose
voxels do not fill a wave. Every output against the oracle, with the bar the
parity tests use."""
import numpy as np
import pytest

import synth
from harness import Run, check_backward, check_forward, is_boxed, log, masked_cotangents, with_long_lists

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("per_cell", [(1, 1, 1), (2, 2, 2), (3, 2, 3), (4, 4, 4), (5, 13, 1), (9, 4, 4)])
def test_grid_cells_of_any_voxel_count(per_cell):
    g = synth.random_gaussians(121, 700, log_mu=np.log(0.06), log_sd=0.5)
    cells = (5, 4, 3)
    dims = tuple(c * r for c, r in zip(cells, per_cell))
    log(f"case grid cells of {per_cell} voxels")
    r = Run(g, cells, "grid", dims=dims)
    phi, inf = r.forward()
    check_forward(r, phi, inf, label=f"{dims}")


def cell_points(rng, cell, cells, n):
    """n points of a cell, some on its faces and quarters."""
    u = rng.random((n, 3))
    snap = rng.random((n, 3)) < 0.05
    u = np.where(snap, np.round(u * 8) / 8, 0.001 + 0.998 * u)
    u = np.clip(u, 0.0, 0.9999)
    return (np.asarray(cell) + u) / np.asarray(cells)


@pytest.mark.parametrize("counts", [
    (0, 1, 3, 4, 31, 63, 64, 700),            # sparse layouts beside dense items
    (65, 127, 128, 191, 192, 193, 319, 320),  # items, and the first boxes
    (321, 383, 385, 577, 1024, 1025, 1100, 1535),
    (1536, 1537, 2049, 3000, 64, 64, 1, 0),   # the finest boxes
])
def test_boxed_launch_at_its_counts(counts):
    rng = np.random.default_rng(sum(counts))
    cells = (2, 2, 2)
    g = synth.random_gaussians(122, 900, log_mu=np.log(0.05), log_sd=0.6)
    pts = [cell_points(rng, (k & 1, (k >> 1) & 1, k >> 2), cells, n) for k, n in enumerate(counts)]
    pts.append(np.array([[1.0, 1.0, 1.0], [1.0001, 0.5, 0.5], [0.0, 0.0, 0.0], [-0.1, 0.2, 0.3]]))
    pts = np.concatenate(pts)
    # queries outside the domain bring the launch to the number that is boxed
    pts = np.concatenate([pts, np.full(((1 << 21) - len(pts), 3), 1.5)]).astype(np.float32)
    rng.shuffle(pts)
    log(f"case boxed launch {counts}")
    r = Run(with_long_lists(g), cells, "points", points=pts)
    phi, inf = r.forward()
    assert is_boxed(r)
    ref, _ = check_forward(r, phi, inf, label=f"boxed {counts}")
    gv, gi = synth.random_normal(123, r.nq), synth.random_normal(124, r.nq)
    gv, gi, _ = masked_cotangents(ref, gv, gi)
    sup = np.nonzero(pts[:, 0] < 1.4)[0]
    check_backward(r, r.backward(gv, gi), np.arange(g.n), sup, gv[sup], gi[sup], label="boxed")


def test_boxed_lists_of_many_chunks_and_empty_cells():
    """Lists of more than the 256 records staged at a time, cells without any
    record, and Gaussians whose boxes reach single corners of the cells."""
    rng = np.random.default_rng(125)
    g = synth.random_gaussians(126, 5000, log_mu=np.log(0.02), log_sd=0.8, lo=0.0, hi=0.49)
    pts = np.concatenate([rng.random((3000, 3)) * 0.5, rng.random((2000, 3)), np.full(((1 << 21) - 5000, 3), 1.5)])
    pts = pts.astype(np.float32)
    log("case boxed lists")
    # long lists in the half x < 0.5 only
    r = Run(with_long_lists(g, 520, (0.25, 0.5, 0.5), (0.05, 0.6, 0.6)), (4, 4, 4), "points", points=pts)
    per = np.diff(r.index_arrays()[2].astype(np.int64))
    assert (per == 0).any() and (per > 3 * 256).any()
    phi, inf = r.forward()
    assert is_boxed(r)
    check_forward(r, phi, inf, label="boxed lists")


def test_boxed_sums_do_not_depend_on_the_batch():
    """A query's sums are formed from its cell's list alone: two batches of one
    level (1,536 queries a cell or more) give the same bits."""
    g = synth.random_gaussians(127, 14000, log_mu=np.log(0.04), log_sd=0.7)
    pts = synth.random_points(128, 5000000)
    log("case boxed batches")
    n = 2200000
    a = Run(g, (4, 4, 4), "points", points=pts)
    b = Run(g, (4, 4, 4), "points", points=pts[:n])
    pa, ia = a.forward()
    pb, ib = b.forward()
    assert is_boxed(a) and is_boxed(b)
    np.testing.assert_array_equal(pa[:n].view(np.uint32), pb.view(np.uint32))
    np.testing.assert_array_equal(ia[:n].view(np.uint32), ib.view(np.uint32))
