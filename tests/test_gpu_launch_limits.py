"""Calls whose blocks do not fit one launch (HIP: fewer than 2^32 threads)."""
import numpy as np
import pytest
import torch

from paper_2511_11078_amd import synth
from paper_2511_11078_amd.ops import Context

from gpu_helpers import rel_l2, say, to_gpu, to_np

pytestmark = pytest.mark.gpu


def _row(w, u, v, pitch, C, centre):
    """One view of one row of C columns, `centre` along u from the origin."""
    return synth.Geometry("parallel", 1, 1, C, np.concatenate([w, centre * u, pitch * u, v])[None].astype(np.float32))


def test_network_forward_of_more_than_one_launch():
    """One row of 16 x 2^24 + 40 columns, a block of 256 threads per 16 of
    them, is four blocks more than one launch takes.  The volume lies before
    its last 4 million columns: those are compared with a row of every 512th
    of them, the others see nothing.  The rows' FP32 centres and pitches put a
    line up to 6e-5 of a coefficient's width apart (335 of them times 2^-24,
    twice, and the centre's own rounding); sums change by no more than their
    own size per such width, and 5e-4 leaves eight times that."""
    C, Cs, step, pitch = 16 * 2**24 + 40, 8192, 512, 2.5e-6
    say(f"network forward, one row of {C} columns")
    w = np.array([1.0, 0.3, 0.2]) / np.linalg.norm([1.0, 0.3, 0.2])
    u, v = synth.detector_frame(w)
    centre = -pitch * (C - 1) / 2 + 4.0  # the last column is 4 beyond the volume's centre
    wide = _row(w, u, v, pitch, C, centre)
    few = _row(w, u, v, pitch * step, Cs, centre + pitch * ((C - 1) / 2 - step * (Cs - 1) / 2))
    c = to_gpu(np.random.default_rng(530).uniform(0.2, 1.0, (4, 5, 6)).astype(np.float32))
    ctx = Context(1, "mlp", 0)
    got, want = ctx.project(c, wide).flatten(), to_np(ctx.project(c, few)).ravel()
    ctx.close()
    e = rel_l2(to_np(got[C - 1 - step * (Cs - 1)::step]), want)
    say(f"  rel-L2 {e:.3e}, non-zero {np.count_nonzero(want)} of {Cs}")
    assert np.count_nonzero(want) > 1000 and e <= 5e-4
    assert int(torch.count_nonzero(got[:C - step * Cs])) == 0


@pytest.mark.parametrize("form", ["quad", "pair"])
def test_forward_of_more_than_2_24_slots(form):
    """Two views of one row of 2^23 + 1 tiles: more than 2^24 blocks, so one
    launch per view.  Equal to the views by themselves."""
    C = 16 * 2**23 + 16
    say(f"{form} forward, two views of one row of {C} columns")
    vecs = []
    for k, w in enumerate(([1.0, 0.3, 0.2], [0.2, -1.0, 0.4])):
        w = np.asarray(w) / np.linalg.norm(w)
        u, v = synth.detector_frame(w)
        vecs.append(_row(w, u, v, 5.0e-7, C, 3.0 * k).vecs)
    geom = synth.Geometry("parallel", 2, 1, C, np.concatenate(vecs))
    c = to_gpu(np.random.default_rng(531).uniform(0.2, 1.0, (4, 5, 6)).astype(np.float32))
    ctx = Context(1, form, 0)
    out = torch.full((2, 1, C), float("nan"), device="cuda")
    ctx.project(c, geom, out)
    one = torch.empty((1, 1, C), device="cuda")
    for k in range(2):
        ctx.project(c, geom.subset_views(k, k + 1), one)
        assert int(torch.count_nonzero(one)) > 1000
        assert torch.equal(out[k], one[0])
    ctx.close()
