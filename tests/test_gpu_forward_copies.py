"""The two padded copies of the quadrature forward: which are made, and that
one at a time gives the bits of both."""
import numpy as np
import pytest
import torch

from paper_2511_11078_amd import synth
from paper_2511_11078_amd.ops import Context

from gpu_helpers import say, to_gpu

pytestmark = pytest.mark.gpu


def _walks_x(geom):
    """The kernel's rule, restated in FP64: the detector direction nearest x
    is nearer to it than the one nearest z is to z, and x is contracted first
    (central ray not within 15 degrees of x, nor 15 to 35 degrees from y)."""
    out = []
    for e in np.asarray(geom.vecs, dtype=np.float64).reshape(-1, 12):
        d = np.abs(e[3:6] - e[0:3] if geom.kind == "cone" else e[0:3])
        u, v = e[6:9] / np.linalg.norm(e[6:9]), e[9:12] / np.linalg.norm(e[9:12])
        hi, lo = max(d[0], d[1]), min(d[0], d[1])
        t15, t35 = np.tan(np.deg2rad([15, 35]))
        yfirst = d[2] < hi and (lo < t15 * hi if d[0] >= d[1] else t15 * hi <= lo < t35 * hi)
        out.append(not yfirst and max(abs(u[0]), abs(v[0])) > max(abs(u[2]), abs(v[2])))
    return out


@pytest.mark.parametrize("n", [0, 3])
def test_circular_trajectory_holds_one_copy(n):
    """A circular trajectory about z walks the z-fastest copy only: the
    context's scratch is that one (200^3: 33 to 36 MB), not two."""
    say(f"one copy n={n}")
    dims = (200, 200, 200)
    geom = synth.cone_circular_geometry(4, 40, 40, src_radius=600.0, src_det=900.0, angle0=0.2)
    assert not any(_walks_x(geom))
    c = torch.zeros(dims[::-1], device="cuda")
    out = torch.empty((geom.n_views, geom.det_rows, geom.det_cols), device="cuda")
    warm = Context(n, "quad", 0)
    warm.project(c[:8, :8, :8].contiguous(), geom, out)
    torch.cuda.synchronize()
    ctx = Context(n, "quad", 0)
    free = torch.cuda.mem_get_info()[0]
    ctx.project(c, geom, out)
    torch.cuda.synchronize()
    took = free - torch.cuda.mem_get_info()[0]
    copy = 4 * (200 + 2 * (n + 1)) ** 3
    say(f"  scratch {took / 1e6:.1f} MB, one copy {copy / 1e6:.1f} MB")
    assert took < 1.5 * copy
    ctx.close()
    warm.close()


@pytest.mark.parametrize("n", [0, 1, 2, 3])
@pytest.mark.parametrize("views", [40, 300])
def test_one_copy_at_a_time(n, views):
    """40 views of 2 x 3 tiles (four lanes a line) and 300 (a line per lane),
    over both copies, with a scratch limit that leaves room for one."""
    say(f"one copy at a time n={n} views={views}")
    dims = (14, 11, 9)
    geom = synth.parallel_geometry(synth.uniform_directions(views, seed=450), 20, 35, pitch=0.6)
    side = _walks_x(geom)
    assert any(side) and not all(side)
    c = to_gpu(np.random.default_rng(451).standard_normal(dims[::-1]).astype(np.float32))
    two, one = Context(n, "quad", 0), Context(n, "quad", 0)
    one.set_scratch_limit(1)
    want = two.project(c, geom)
    got = one.project(c, geom, torch.full_like(want, float("nan")))
    assert torch.equal(got, want)
    two.close()
    one.close()


@pytest.mark.parametrize("n", [0, 2, 3])
@pytest.mark.parametrize("pitch", [0.8, 1.9])
def test_shared_lines_on_large_copies(n, pitch):
    """140^3 (a copy above 2^21 floats), views of 4 x 5 tiles with dense and
    with sparse lines: all 27 of them (540 tiles) and one at a time, on either
    side of the shared-line rule where it has one between them.  Equal bits."""
    say(f"shared lines on a large copy n={n} pitch={pitch}")
    dims = (140, 139, 138)
    geom = synth.parallel_geometry(synth.uniform_directions(27, seed=460), 60, 77, pitch=pitch)
    c = torch.randn(dims[::-1], generator=torch.Generator("cuda").manual_seed(461), device="cuda")
    ctx = Context(n, "quad", 0)
    whole = ctx.project(c, geom)
    parts = [ctx.project(c, geom.subset_views(v, v + 1)) for v in range(geom.n_views)]
    assert torch.equal(whole, torch.cat(parts))
    ctx.close()
