"""GPU parity where rows are whole 64-cell segments (nx % 64 == 0), the layout by
segments of the advection sweeps: alone, and in batches whose boxes all have such
rows (one box with other rows gives the whole batch the flat layout).

The x-sweep takes a row by one wavefront up to `chunk` segments, and above that by
several wavefronts that exchange their segments' ends through LDS: 32 segments
(2048 cells) in the plain call, 8 (512 cells) in a batch tuned to chunk 8. With a
tuning a fixed grid of workgroups walks the work items, so that a workgroup takes
several items in turn, among them such of an odd number of positions.

Bars: 1e-12 to the oracle, the volume-fraction tolerance of the other advection
tests; a batch bit-identical to plain calls."""
import numpy as np
import pytest

import oracle
from gpu_util import note, require_gpu
from paper_2407_07463_amd import synth

pytestmark = pytest.mark.gpu
TOL = 1e-12


@pytest.fixture(scope="module")
def ctx():
    require_gpu()
    from paper_2407_07463_amd import vofmt

    c = vofmt.Context(0)
    yield c
    c.close()


def _random(shape, ntr, seed):
    nz, ny, nx = shape
    rng = synth.Splitmix64(seed)
    v = rng.uniform(ntr * nx * ny * nz).reshape((ntr,) + shape)
    c = np.where(v < 0.3, 0.0, np.where(v > 0.7, 1.0, (v - 0.3) / 0.4))
    return c, [(rng.uniform(nx * ny * nz).reshape(shape) - 0.5) * 0.9 for _ in range(3)]


def _dev(*arrays):
    import torch

    return [torch.from_numpy(a).to("cuda:0") for a in arrays]


def _batch_like_plain(ctx, sizes, step0, nsteps, tuning, seed):
    import torch

    boxes = [_dev(c, *s) for c, s in (_random(shape, ntr, seed + i) for i, (shape, ntr) in enumerate(sizes))]
    alone = [b[0].clone() for b in boxes]
    for a, b in zip(alone, boxes):
        ctx.advect(a, *b[1:], step0=step0, nsteps=nsteps)
    ctx.advect_batched([tuple(b) for b in boxes], step0=step0, nsteps=nsteps, tuning=tuning)
    torch.cuda.synchronize()
    for size, a, b in zip(sizes, alone, boxes):
        assert torch.equal(a, b[0]), size


@pytest.mark.parametrize("sizes,tuning", [
    ([((33, 40, 576), 4)], (8, 1)),                         # 600 items of 8 planes or 1, 256 workgroups
    ([((1, 300, 576), 3)], (8, 1)),                         # one plane: every item an odd number of positions
    ([((17, 50, 1088), 2), ((9, 30, 576), 3)], (16, 1)),    # rows above and below the chunk's segments
])
@pytest.mark.parametrize("step0", [0, 1, 2])
def test_split_rows_of_a_fixed_grid(ctx, sizes, tuning, step0):
    """Items of the LDS x-sweep follow one another in a workgroup."""
    note(f"batched split rows {sizes} tuning={tuning} step0={step0}")
    _batch_like_plain(ctx, sizes, step0, 1, tuning, 811)


@pytest.mark.parametrize("step0", [0, 1, 2])
@pytest.mark.parametrize("shape,ntr", [((4, 6, 2112), 1), ((3, 5, 2112), 3), ((5, 3, 2176), 4), ((2, 4, 2112), 5),
                                       ((4, 2, 2624), 7), ((5, 9, 2048), 3), ((9, 8, 576), 7), ((17, 33, 320), 5)])
def test_rows_of_whole_segments(ctx, shape, ntr, step0):
    """Above and at 2048 cells (several wavefronts a row, one), in groups of 1 to 4 tracers."""
    import torch

    c, s = _random(shape, ntr, 41 + sum(shape))
    note(f"advect whole segments {shape} ntr={ntr} step0={step0}")
    tc, *ts = _dev(c, *s)
    ctx.advect(tc, *ts, step0=step0, nsteps=2)
    torch.cuda.synchronize()
    assert np.abs(tc.cpu().numpy() - oracle.advect(c, *s, step0, 2)).max() <= TOL


@pytest.mark.parametrize("tuning", [None, (8, 1), (8, 16), (16, 2), (32, 4), (64, 8), (64, 32)])
@pytest.mark.parametrize("step0,nsteps", [(0, 1), (1, 2), (5, 3)])
def test_batch_of_whole_segments(ctx, tuning, step0, nsteps):
    """Rows of 1 to 33 segments and groups of 1 to 4 tracers in one batch by segments."""
    sizes = [((20, 24, 64), 3), ((9, 33, 128), 5), ((12, 10, 576), 4), ((5, 7, 320), 7), ((6, 5, 2112), 2), ((3, 4, 192), 1)]
    note(f"batch of whole segments tuning={tuning} step0={step0} nsteps={nsteps}")
    _batch_like_plain(ctx, sizes, step0, nsteps, tuning, 907)
