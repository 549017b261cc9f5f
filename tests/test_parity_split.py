"""GPU parity of the advection against the CPU oracle where the split of the
work over wavefronts changes: the marching chunk falls from 32 to 16, 8 and 4
with the number of wavefronts of a sweep, and the initial scan's span with the
number of tracer-cells. Bar: 1e-12, the volume-fraction tolerance of the
other advection tests (one or two steps of fields whose values are O(1))."""
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


@pytest.mark.parametrize("shape,ntr,step0,nsteps", [
    ((5, 4, 64), 1, 0, 1), ((9, 33, 65), 1, 1, 2),  # chunk 4: whole chunks, remainders of 1
    ((1, 1, 7), 1, 0, 1), ((4, 3, 1), 2, 2, 2),     # single rows and columns
    ((37, 40, 257), 3, 2, 2),                       # 5 segments a row: chunk 8
    ((8, 31, 515), 2, 0, 2),                        # 9 segments: chunk 16
    # tracer groups of even sizes: 3 + 2, 4 + 3, 4 + 3 + 3 + 3
    ((9, 10, 70), 5, 0, 1), ((13, 8, 66), 7, 1, 2), ((6, 9, 65), 13, 2, 1),
    ((300, 150, 128), 2, 0, 1),                     # chunk 8 from the number of wavefronts
    ((300, 300, 128), 1, 1, 1),                     # chunk 16
    ((129, 258, 320), 4, 2, 1),                     # chunk 16 to 32, a scan span that does not divide the field
])
def test_work_split(ctx, shape, ntr, step0, nsteps):
    import torch

    c, s = _random(shape, ntr, 31 + sum(shape))
    note(f"advect split {shape} ntr={ntr} step0={step0} nsteps={nsteps}")
    tc = torch.from_numpy(c).to("cuda:0")
    ctx.advect(tc, *[torch.from_numpy(a).to("cuda:0") for a in s], step0=step0, nsteps=nsteps)
    torch.cuda.synchronize()
    assert np.abs(tc.cpu().numpy() - oracle.advect(c, *s, step0, nsteps)).max() <= TOL
