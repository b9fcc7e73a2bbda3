"""The quadrature scratch: its growth policy on the host (csrc/ss_scratch.hpp,
HIP-free, compiled with g++), and a forward captured on a context whose
scratch holds one padded copy but not the two it would like."""
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_growth_policy(tmp_path):
    exe = tmp_path / "scratch_test"
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-fsanitize=address,undefined",
                    "-I", os.path.join(ROOT, "paper_2511_11078_amd", "csrc"),
                    os.path.join(ROOT, "tests", "host", "scratch_test.cpp"), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
    assert "all checks passed" in r.stdout


@pytest.mark.gpu
def test_forward_captured_after_an_adjoint():
    """Degree 0, 20 x 20 x 1: the adjoint leaves a table of 3 x 3 bricks of 256
    floats, 2,304; one padded copy takes 22 x 22 x 3 = 1,452.  The capture
    allocates, frees and waits for nothing, and every replay gives the eager
    result's bits."""
    import torch

    from paper_2511_11078_amd import synth
    from paper_2511_11078_amd.ops import Context
    from gpu_helpers import say, to_gpu

    say("forward captured after an adjoint")
    dims = (20, 20, 1)
    vecs = []
    for w, roll in (([0.1, -0.2, 1.0], 0.0), ([0.3, 1.0, -0.2], 0.3), ([0.0, 0.01, 1.0], np.pi / 2)):
        w = np.asarray(w) / np.linalg.norm(w)
        u, v = synth.detector_frame(w)
        c, s = np.cos(roll), np.sin(roll)
        vecs.append(np.concatenate([w, np.zeros(3), c * u + s * v, c * v - s * u]))
    geom = synth.Geometry("parallel", len(vecs), 17, 24, np.asarray(vecs, dtype=np.float32))
    rng = np.random.default_rng(540)
    y = to_gpu(rng.standard_normal((geom.n_views, geom.det_rows, geom.det_cols)).astype(np.float32))
    vols = [to_gpu(rng.standard_normal(dims[::-1]).astype(np.float32)) for _ in range(3)]
    eager = Context(0, "quad", 0)
    want = [eager.project(v, geom) for v in vols]
    ctx = Context(0, "quad", 0)
    ctx.backproject(y, geom, dims)
    torch.cuda.synchronize()
    c = vols[0].clone()
    out = torch.zeros_like(want[0])
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        ctx.project(c, geom, out)
    for k in (1, 2, 0, 1):
        c.copy_(vols[k])
        out.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want[k])
        assert torch.equal(eager.project(vols[k], geom), want[k])
    ctx.close()
    eager.close()
