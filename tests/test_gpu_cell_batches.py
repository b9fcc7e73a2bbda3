"""View batches of the quadrature adjoint's cell gather against the FP64 oracle.

A block takes its views in batches: up to 8 consecutive views whose line
rectangles together fit half of its line table, a larger view alone in
segments, per-view constants for 64 views at a time; a table with an
axis-parallel line takes another slab test; at degrees 2 and 3 volumes of up
to 256 bricks share each cell's moments among waves, of larger ones a thread
holds them all.  The cases sit on the edges of those rules; the bar is the quadrature form's (relative L2 1e-5 for
FP32 arithmetic, 1e-4 for degree 0, whose outputs jump where a line runs
within rounding of a voxel face).
"""
import numpy as np
import pytest

import oracle
from paper_2511_11078_amd import synth
from paper_2511_11078_amd.ops import Context

from gpu_helpers import rel_l2, say, to_gpu, to_np

pytestmark = pytest.mark.gpu


def _tilted(views, pitches, shift, seed):
    """Parallel views with a pitch of their own each; every third one's
    detector moved by `shift` pixels along its columns."""
    vecs = []
    for k, w in enumerate(synth.uniform_directions(views, seed=seed)):
        u, v = synth.detector_frame(w)
        p = pitches[k % len(pitches)]
        vecs.append(np.concatenate([w, (shift * p if k % 3 == 0 else 0.0) * u, p * u, p * v]))
    return np.asarray(vecs, dtype=np.float32)


CASES = {
    # name: (views, rows, cols, pitches, detector shift)
    "one_view": (1, 9, 11, [1.0], 0.0),
    "seven_views_one_pixel": (7, 1, 1, [1.0], 0.0),
    "records_of_65_views": (65, 6, 7, [1.0], 0.0),
    "records_of_129_views_some_missing": (129, 5, 6, [1.1], 40.0),
    # 8 x 8 x 4 cells span about 12 x 12 pixels at pitch 1: from batches of
    # several views, over one view per batch, to views in segments, in turn
    "batches_and_segments_in_turn": (22, 60, 90, [1.0, 0.62, 0.5, 0.2], 0.0),
    "wider_than_a_run": (5, 4, 300, [0.11], 0.0),
}
VOLUMES = {"small": (11, 9, 6), "large": (61, 53, 25)}  # 12 and 392 bricks of cells at degree 3


def _adjoint_error(n, geom, dims, seed):
    y = np.random.default_rng(seed).standard_normal((geom.n_views, geom.det_rows, geom.det_cols)).astype(np.float32)
    ctx = Context(n, "quad", 0)
    got = to_np(ctx.backproject(to_gpu(y), geom, dims))
    ctx.close()
    coefs = synth.sample_indices(int(np.prod(dims)), 600, seed=seed + 1)
    want = oracle.backproject_subset(y, geom, dims, n, coefs=coefs)
    assert np.abs(want).max() > 0
    return rel_l2(got.ravel()[coefs], want)


@pytest.mark.parametrize("n", [0, 1, 2, 3])
@pytest.mark.parametrize("case", list(CASES))
@pytest.mark.parametrize("volume", list(VOLUMES))
def test_view_batches(n, case, volume):
    say(f"cell gather {case} {volume} n={n}")
    views, R, C, pitches, shift = CASES[case]
    if volume == "large":  # as many pixels per cell, over more of the volume
        R, C = max(R, 24), max(C, 33)
    geom = synth.Geometry("parallel", views, R, C, _tilted(views, pitches, shift, seed=300 + n))
    e = _adjoint_error(n, geom, VOLUMES[volume], 310 + n)
    say(f"  rel-L2 {e:.3e}")
    assert e <= (1e-5 if n > 0 else 1e-4)


@pytest.mark.parametrize("n", [0, 1, 2, 3])
@pytest.mark.parametrize("volume", list(VOLUMES))
def test_axis_parallel_lines_in_some_batches(n, volume):
    """Groups of views whose lines all, some or none run parallel to an axis,
    in and beside the knot planes."""
    say(f"cell gather axis-parallel lines {volume} n={n}")
    dirs = list(synth.great_circle_plus_tilts(7, 9, seed=320)) + [[1, 0, 0], [0, 1, 0], [0, 0, 1]]
    dirs += list(synth.uniform_directions(11, seed=321)) + [[0, 0.6, 0.8], [0.6, 0, 0.8]]
    geom = synth.parallel_geometry(np.asarray(dirs, dtype=np.float64), 23, 26)
    # off the voxel faces at degree 0, where a line in a face meets no voxel
    if n == 0:
        geom.vecs[:, 3:6] += np.float32(0.17)
    e = _adjoint_error(n, geom, VOLUMES[volume], 330 + n)
    say(f"  rel-L2 {e:.3e}")
    assert e <= (1e-5 if n > 0 else 1e-4)


@pytest.mark.parametrize("n", [0, 1, 2, 3])
@pytest.mark.parametrize("dims", [(1, 1, 1), (5, 5, 1), (6, 6, 2), (13, 5, 9), (64, 58, 37)])
@pytest.mark.parametrize("limit", [0, 1])
def test_parts_of_blocks(n, dims, limit):
    """A coefficient's sum over the blocks of cells its support meets: one
    block, exactly one at degree 3, one cell more, odd counts, and many, in
    one pass and in z-chunks (the smallest scratch), on every coefficient."""
    say(f"parts of blocks n={n} {dims} limit {limit}")
    if n == 1 and dims == (1, 1, 1):
        pytest.skip("all ten lines that meet it graze its support (footprints below 4.3e-5 of a unit): "
                    "the one value there is, 1e-5, is below what a bar relative to it can hold in FP32")
    geom = synth.parallel_geometry(synth.uniform_directions(3, seed=340), 40, 44, pitch=2.1)
    y = np.random.default_rng(341 + n).standard_normal((3, 40, 44)).astype(np.float32)
    ctx = Context(n, "quad", 0)
    ctx.set_scratch_limit(limit)
    got = to_np(ctx.backproject(to_gpu(y), geom, dims))
    ctx.close()
    want = oracle.backproject_subset(y, geom, dims, n)
    e = rel_l2(got.ravel(), np.asarray(want).ravel())
    say(f"  rel-L2 {e:.3e}")
    assert e <= (1e-5 if n > 0 else 1e-4)


FINE = {
    # name: (views, rows, cols, pitches, detector shift)
    "rows_wider_than_64_in_batches": (9, 1, 410, [0.12, 0.9, 0.06], 0.0),
    "columns_taller_than_64_in_batches": (9, 270, 1, [0.1, 0.2], 0.0),
    "queued_segments": (7, 70, 90, [0.25, 0.16], 0.0),
    # a cell's pixels in a row: 61 still go into a run, the next pitch not
    "edge_of_a_run": (8, 5, 700, [0.03, 0.025, 0.02, 1.0, 0.012], 0.0),
    "queued_and_direct_in_turn": (9, 33, 120, [0.2, 0.015, 0.05], 0.0),
}


@pytest.mark.parametrize("n", [0, 1, 2, 3])
@pytest.mark.parametrize("case", list(FINE))
def test_fine_pixels(case, n):
    """Views whose rectangle on a brick is larger than the line table's half,
    or than a run of the queue, before and after views that fit."""
    views, R, C, pitches, shift = FINE[case]
    say(f"cell batches, fine pixels {case} n={n}")
    geom = synth.Geometry("parallel", views, R, C, _tilted(views, pitches, shift, seed=330))
    dims = VOLUMES["small"] if case != "queued_segments" else (19, 18, 33)
    e = _adjoint_error(n, geom, dims, 331)
    say(f"  rel-L2 {e:.3e}")
    assert e <= (1e-5 if n > 0 else 1e-4)


@pytest.mark.parametrize("n", [0, 1, 2, 3])
@pytest.mark.parametrize("dims", [(1, 2, 3), (5, 13, 4), (9, 8, 17), (52, 44, 61)])
def test_parts_are_summed_once(n, dims):
    """The sums over a block's cells and over the blocks of a coefficient load
    every part they might need and add 0 for those that are not there: every
    coefficient of volumes around the blocks' edges against the oracle, and
    non-finite parts stay where they belong."""
    say(f"parts of blocks n={n} {dims}")
    geom = synth.Geometry("parallel", 3, 30, 31, _tilted(3, [max(dims) / 20.0], 0.0, seed=350))
    y = np.random.default_rng(351).standard_normal((3, 30, 31)).astype(np.float32)
    ctx = Context(n, "quad", 0)
    got = to_np(ctx.backproject(to_gpu(y), geom, dims))
    want = oracle.backproject_subset(y, geom, dims, n)
    assert np.abs(want).max() > 0
    e = rel_l2(got, want)
    say(f"  rel-L2 {e:.3e}")
    assert e <= (1e-5 if n > 0 else 1e-4)
    # one infinite pixel: only coefficients that its line meets (by the
    # oracle) may differ from the finite result
    y[1, 15, 16] = 0.0
    base = to_np(ctx.backproject(to_gpu(y), geom, dims))
    y[1, 15, 16] = np.inf
    inf = to_np(ctx.backproject(to_gpu(y), geom, dims))
    ctx.close()
    one = np.zeros_like(y)
    one[1, 15, 16] = 1.0
    met = oracle.backproject_subset(one, geom, dims, n).reshape(got.shape) != 0
    h = np.pad(met, n + 1)
    near = np.zeros_like(met)
    for dz in range(2 * n + 3):
        for dy in range(2 * n + 3):
            for dx in range(2 * n + 3):
                near |= h[dz:dz + met.shape[0], dy:dy + met.shape[1], dx:dx + met.shape[2]]
    assert np.array_equal(inf[~near], base[~near])
    assert met.any() and not np.isfinite(inf[met]).all()
