"""Rules of the quadrature forward's launch, against the FP64 oracle and
against each other.

A launch of few 16 x 16-pixel tiles (512, 320, 768, 1536 at degrees 0 to 3)
shares each line among four lanes; a view is walked over a copy of the coefficients with z or with
x fastest, its lanes along the detector direction nearest that axis; copies
above 4 GiB take 64-bit offsets.  None of it may change a sum: launches that
fall on either side of a rule give equal bits, and the bar against the
oracle is the quadrature form's (relative L2 1e-5, 1e-4 for degree 0).
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2511_11078_amd import synth
from paper_2511_11078_amd.ops import Context, project_noalloc

from gpu_helpers import rel_l2, say, to_gpu, to_np

pytestmark = pytest.mark.gpu


def _views(dirs, rolls, R, C, pitch=1.0):
    """Parallel views whose detector is rolled about the ray."""
    vecs = []
    for w, roll in zip(dirs, rolls):
        w = np.asarray(w, dtype=np.float64) / np.linalg.norm(w)
        u, v = synth.detector_frame(w)
        c, s = np.cos(roll), np.sin(roll)
        vecs.append(np.concatenate([w, np.zeros(3), pitch * (c * u + s * v), pitch * (c * v - s * u)]))
    return synth.Geometry("parallel", len(vecs), R, C, np.asarray(vecs, dtype=np.float32))


@pytest.mark.parametrize("n", [0, 1, 2, 3])
@pytest.mark.parametrize("R,C", [(1, 1), (3, 17), (16, 16), (33, 5)])
def test_copies_and_lane_directions(n, R, C):
    """Rays along every axis and between, detectors rolled by 0, 45 and 90
    degrees: both copies, lanes along rows and along columns."""
    say(f"forward walk n={n} detector {R}x{C}")
    dims = (14, 11, 9)
    dirs = [[1, 0, 0], [0, 1, 0], [0, 0, 1], [1, 0.2, 0.1], [0.3, 1, -0.2], [0.1, -0.2, 1], [1, 1, 1], [-0.5, 0.4, -1]]
    dirs = [np.asarray(d, dtype=np.float64) + 1e-3 * k for k, d in enumerate(dirs)] + [[0, 0, 1], [0, 1, 0]]
    rolls = [0.0, np.pi / 2, np.pi / 4, 0.3, np.pi / 2, np.pi / 2, 1.0, 0.0, np.pi / 2, 0.0]
    geom = _views(dirs, rolls, R, C, pitch=0.77)
    c = np.random.default_rng(400 + n).standard_normal(dims[::-1]).astype(np.float32)
    ctx = Context(n, "quad", 0)
    got = ctx.project(to_gpu(c), geom)
    one = torch.cat([ctx.project(to_gpu(c), geom.subset_views(k, k + 1)) for k in range(geom.n_views)])
    assert torch.equal(got, one)
    assert torch.equal(got, project_noalloc(to_gpu(c), geom, degree=n))
    ctx.close()
    want = oracle.project(c, geom, n)
    e = rel_l2(to_np(got), want)
    say(f"  rel-L2 {e:.3e}")
    assert e <= (1e-5 if n > 0 else 1e-4)


@pytest.mark.parametrize("n", [0, 1, 2, 3])
def test_shared_lines_equal_unshared(n):
    """4098 tiles in one launch (a line per lane), and in launches of at most 318 (four lanes)."""
    say(f"shared lines n={n}")
    dims = (10, 9, 8)
    views, R, C = 683, 20, 35  # 2 x 3 tiles of 16 x 16 pixels a view: 4098 tiles; 53 views: 318
    geom = synth.parallel_geometry(synth.uniform_directions(views, seed=410), R, C, pitch=0.5)
    c = to_gpu(np.random.default_rng(411).standard_normal(dims[::-1]).astype(np.float32))
    ctx = Context(n, "quad", 0)
    whole = ctx.project(c, geom)
    parts = [ctx.project(c, geom.subset_views(v, min(v + 53, views))) for v in range(0, views, 53)]
    assert torch.equal(whole, torch.cat(parts))
    ctx.close()


def test_copy_above_4_gib():
    """A padded copy of more than 2^30 coefficients, non-zero only near its
    far end, rays along x and along z."""
    dims = (1040, 1032, 1000)
    say(f"forward walk over {dims}")
    c = np.zeros(dims[::-1], dtype=np.float32)
    c[-12:, -20:, -24:] = np.random.default_rng(420).standard_normal((12, 20, 24)).astype(np.float32)
    vecs = []
    for w, p in (([1.0, 0.003, -0.002], (0.0, 500.0, 490.0)), ([0.002, -0.004, 1.0], (505.0, 502.0, 0.0))):
        u, v = synth.detector_frame(np.asarray(w) / np.linalg.norm(w))
        vecs.append(np.concatenate([w, p, u, v]))
    geom = synth.Geometry("parallel", 2, 24, 26, np.asarray(vecs, dtype=np.float32))
    ctx = Context(3, "quad", 0)
    got = to_np(ctx.project(to_gpu(c), geom))
    ctx.close()
    want = oracle.project(c, geom, 3)
    e = rel_l2(got, want)
    say(f"  rel-L2 {e:.3e}")
    assert np.abs(want).max() > 0 and e <= 1e-5


@pytest.mark.parametrize("n", [2, 3])
@pytest.mark.parametrize("dims", [(310, 320, 310), (340, 330, 310)])
def test_lane_tiles(n, dims):
    """Copies just below and above 2^25 floats, walked in waves of 8 x 8 and
    of 16 x 4 pixels: 2100 tiles in one launch, and 420 a launch (four lanes
    a line).  No line's sum depends on its lane."""
    say(f"lane tiles n={n} {dims}")
    geom = synth.parallel_geometry(synth.uniform_directions(5, seed=430), 330, 310, pitch=1.3)
    c = to_gpu(np.random.default_rng(431).standard_normal(dims[::-1]).astype(np.float32))
    ctx = Context(n, "quad", 0)
    whole = ctx.project(c, geom)
    parts = [ctx.project(c, geom.subset_views(v, v + 1)) for v in range(5)]
    assert torch.equal(whole, torch.cat(parts))
    ctx.close()


@pytest.mark.parametrize("views,R,C", [(2105, 9, 13), (1, 740, 725), (9, 260, 270), (23, 33, 500)])
def test_every_tile_of_every_view(views, R, C):
    """More than 2048 tiles, dealt to the XCDs in items of 2 x 2 tiles of up
    to eight views: fewer tiles than an item, one view, a last item of one
    view, odd tile counts.  Every pixel is written, by its own line."""
    say(f"tiles of {views} views {R}x{C}")
    dims = (12, 10, 9)
    geom = synth.parallel_geometry(synth.uniform_directions(views, seed=440), R, C, pitch=14.0 / max(R, C))
    c = np.random.default_rng(441).uniform(0.5, 1.0, dims[::-1]).astype(np.float32)
    ctx = Context(1, "quad", 0)
    out = torch.full((views, R, C), float("nan"), device="cuda")
    got = to_np(ctx.project(to_gpu(c), geom, out=out))
    ctx.close()
    want = oracle.project(c, geom, 1)
    e = rel_l2(got, want)
    say(f"  rel-L2 {e:.3e}")
    assert np.isfinite(got).all() and e <= 1e-5
