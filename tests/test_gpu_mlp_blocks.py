"""Block shapes of the network form against brute-force pair sums.

Forward blocks share 8 x 4 lines, or 4 x 4 for up to 1024 tiles of 16 x 16
pixels, each group of so many lanes some of their slabs; adjoint blocks a brick of 4 x 4 x 4 coefficients, each wave every
fourth candidate pixel of them, or, for more than 768 bricks of
8 x 8 x 4, one such brick with a coefficient per thread.  Volumes and
detectors at the edges of those shapes; the bars are those of the pair
enumeration tests (2e-5 forward, 3e-5 for the adjoint of a noise sinogram).
"""
import numpy as np
import pytest

from paper_2511_11078_amd import footprint_net as fn
from paper_2511_11078_amd.ops import Context, default_weights

from gpu_helpers import rel_l2, say, tilted_parallel, to_gpu, to_np
from test_gpu_mlp import _pairs_reference, _pairs_reference_adjoint

pytestmark = pytest.mark.gpu

CASES = {
    # name: (dims, views, rows, cols, pitch)
    "one_coefficient_one_line": ((1, 1, 1), 2, 1, 1, 1.0),
    "one_slab": ((9, 7, 1), 2, 9, 3, 0.9),
    "last_launch_of_16_lines": ((4, 3, 5), 1024, 1, 2, 1.0),   # 1024 tiles
    "first_launch_of_32_lines": ((4, 3, 5), 1025, 2, 1, 1.0),
    "one_candidate_column": ((5, 4, 13), 3, 17, 1, 0.3),
    "brick_edges": ((4, 8, 5), 3, 8, 9, 0.8),
    "segments_of_the_line_table": ((5, 3, 4), 2, 40, 21, 0.25),
    "last_small_brick_volume": ((64, 64, 48), 1, 5, 4, 3.0),   # 8 x 8 x 12 = 768 bricks
    "first_large_brick_volume": ((64, 64, 49), 1, 4, 5, 3.0),  # 832
}


@pytest.mark.parametrize("case", list(CASES))
def test_blocks_match_pair_enumeration(case):
    dims, views, R, C, pitch = CASES[case]
    say(f"network blocks {case} {dims}")
    with open(default_weights(3), "rb") as fh:
        blob = fn.parse_blob(fh.read())
    rng = np.random.default_rng(500)
    geom = tilted_parallel(views, R, C, seed=501, pitch=pitch)
    c = rng.uniform(0.2, 1.0, dims[::-1]).astype(np.float32)
    y = rng.standard_normal((views, R, C)).astype(np.float32)
    ctx = Context(3, "mlp", 0)
    got_f, got_b = to_np(ctx.project(to_gpu(c), geom)), to_np(ctx.backproject(to_gpu(y), geom, dims))
    ctx.close()
    want_f, want_b = _pairs_reference(blob, 3, c, geom), _pairs_reference_adjoint(blob, 3, y, geom, dims)
    ef, eb = rel_l2(got_f, want_f), rel_l2(got_b, want_b)
    say(f"  forward rel-L2 {ef:.3e}, adjoint rel-L2 {eb:.3e}")
    assert np.abs(want_f).max() > 0 and np.abs(want_b).max() > 0
    assert ef <= 2e-5 and eb <= 3e-5


def test_line_sharing_rules_agree():
    """1800 tiles in one launch (32 lines a block) and 900 (16 lines): every
    line of ragged tiles gets its own sum, to the form's bar."""
    say("network forward: 32 and 16 lines a block")
    dims, views = (9, 8, 21), 300
    geom = tilted_parallel(views, 17, 40, seed=510, pitch=0.6)
    c = to_gpu(np.random.default_rng(511).uniform(0.2, 1.0, dims[::-1]).astype(np.float32))
    ctx = Context(3, "mlp", 0)
    whole = to_np(ctx.project(c, geom))
    parts = [to_np(ctx.project(c, geom.subset_views(v, v + 150))) for v in (0, 150)]
    ctx.close()
    e = rel_l2(whole, np.concatenate(parts))
    say(f"  rel-L2 {e:.3e}")
    assert np.abs(whole).max() > 0 and e <= 2e-5


THIN = {
    # name: (dims, views, rows, cols, pitch); patches of 16 or 32 lines of a 16 x 16 tile
    "one_row": ((9, 8, 7), 3, 1, 37, 0.4),
    "one_column": ((9, 8, 7), 3, 37, 1, 0.4),
    "two_rows": ((6, 5, 7), 3, 2, 19, 0.6),
    "two_columns": ((6, 5, 7), 3, 21, 2, 0.6),
    "three_by_three": ((6, 5, 7), 3, 3, 3, 1.5),
    "many_views_of_one_row": ((4, 3, 5), 1030, 1, 5, 1.0),     # more than 1024 tiles
    "many_views_of_two_rows": ((4, 3, 5), 1030, 2, 3, 1.0),    # 32 lines: 2 x 16
    "many_views_of_three_columns": ((4, 3, 5), 1030, 5, 3, 1.0),
    "many_views_of_nine_rows": ((4, 3, 5), 520, 9, 17, 0.5),
}


@pytest.mark.parametrize("case", list(THIN))
def test_patches_of_thin_detectors(case):
    """Detectors of fewer rows or columns than a patch of lines."""
    dims, views, R, C, pitch = THIN[case]
    say(f"network patches {case} {dims}")
    with open(default_weights(3), "rb") as fh:
        blob = fn.parse_blob(fh.read())
    geom = tilted_parallel(views, R, C, seed=520, pitch=pitch)
    c = np.random.default_rng(521).uniform(0.2, 1.0, dims[::-1]).astype(np.float32)
    ctx = Context(3, "mlp", 0)
    got = to_np(ctx.project(to_gpu(c), geom))
    ctx.close()
    want = _pairs_reference(blob, 3, c, geom)
    e = rel_l2(got, want)
    say(f"  rel-L2 {e:.3e}")
    assert np.abs(want).max() > 0 and e <= 2e-5
