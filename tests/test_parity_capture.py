"""Advection calls of an odd number of sweeps inside a HIP graph that the caller
captures: the first time in the context (no memory may be taken during a capture:
the result is copied back) and with the third field copy at hand; replays with
eager calls of other sizes between them, which must not touch what the graph
uses. A batch whose third copies would have to grow past a captured one copies
back as well. Every result is bit-identical to the eager call."""
import numpy as np
import pytest

from gpu_util import note, require_gpu
from paper_2407_07463_amd import synth

pytestmark = pytest.mark.gpu


def _random(shape, ntr, seed):
    import torch

    nz, ny, nx = shape
    rng = synth.Splitmix64(seed)
    v = rng.uniform(ntr * nx * ny * nz).reshape((ntr,) + shape)
    c = np.where(v < 0.3, 0.0, np.where(v > 0.7, 1.0, (v - 0.3) / 0.4))
    s = [(rng.uniform(nx * ny * nz).reshape(shape) - 0.5) * 0.9 for _ in range(3)]
    return [torch.from_numpy(a).to("cuda:0") for a in (c, *s)]


@pytest.mark.parametrize("third", [False, True])
@pytest.mark.parametrize("shape,ntr", [((17, 30, 65), 3), ((12, 20, 128), 2)])
def test_captured_odd_call(shape, ntr, third):
    torch = require_gpu()
    from paper_2407_07463_amd import vofmt

    note(f"captured advection {shape} x {ntr} third={third}")
    ctx = vofmt.Context(0)
    try:
        c0, *s = _random(shape, ntr, 97)
        big, *sb = _random((24, 40, 130), ntr + 1, 98)
        ctx.advect(big.clone(), *sb, step0=0, nsteps=2)  # the other buffers: large enough for all calls here
        eager = vofmt.Context(0)
        want = c0.clone()
        want_big = big.clone()
        eager.advect(want_big, *sb, step0=0, nsteps=1)
        stream = torch.cuda.Stream()
        c = c0.clone()
        torch.cuda.synchronize()
        with torch.cuda.stream(stream):
            ctx.advect(c, *s, step0=0, nsteps=1 if third else 2)  # warm; nsteps 1 takes the third copy
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            ctx.advect(c, *s, step0=0, nsteps=1)
        c.copy_(c0)
        for replay in range(4):
            graph.replay()
            torch.cuda.synchronize()
            eager.advect(want, *s, step0=0, nsteps=1)
            torch.cuda.synchronize()
            assert torch.equal(c, want), replay
            other = big.clone()  # needs a larger third copy than the graph's
            ctx.advect(other, *sb, step0=0, nsteps=1)
            filler = torch.full((big.numel(),), float(replay), dtype=torch.float64, device="cuda:0")
            torch.cuda.synchronize()
            assert torch.equal(other, want_big)
            assert bool((filler == replay).all())
        eager.close()
    finally:
        ctx.close()


@pytest.mark.parametrize("nsteps", [1, 3])
@pytest.mark.parametrize("nx", [65, 128])
def test_batch_copied_back(nx, nsteps):
    torch = require_gpu()
    from paper_2407_07463_amd import vofmt

    note(f"batch copied back nx={nx} nsteps={nsteps}")
    ctx, other = vofmt.Context(0), vofmt.Context(0)
    try:
        c0, *s = _random((9, 10, 33), 1, 5)
        stream = torch.cuda.Stream()
        torch.cuda.synchronize()
        with torch.cuda.stream(stream):
            ctx.advect(c0, *s, step0=0, nsteps=1)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            ctx.advect(c0, *s, step0=0, nsteps=1)
        boxes = [tuple(_random(shape, ntr, 60 + i)) for i, (shape, ntr) in enumerate([((20, 33, nx), 3), ((7, 40, 64), 1)])]
        want = [b[0].clone() for b in boxes]
        for w, b in zip(want, boxes):
            other.advect(w, *b[1:], step0=1, nsteps=nsteps)
        ctx.advect_batched(boxes, step0=1, nsteps=nsteps)
        torch.cuda.synchronize()
        for w, b in zip(want, boxes):
            assert torch.equal(w, b[0])
    finally:
        ctx.close()
        other.close()
