"""GPU parity of the reassignment where drops of different tracers overlap deeply:
cells shared by several drops, inside some of them and on the boundary of others.
Pairs of tracers at every distance below and above the reach, from tiles in LDS
(reach up to 2 and up to 4) and from the list of boundary cells (above, and on
axes no longer than the tile's halo). Bit-exact to the oracle."""
import numpy as np
import pytest

import oracle
from gpu_util import note, require_gpu
from paper_2407_07463_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    require_gpu()
    from paper_2407_07463_amd import vofmt

    c = vofmt.Context(0)
    yield c
    c.close()


def _fields(kind, shape, ntr):
    nz, ny, nx = shape
    rng = synth.Splitmix64(sum(shape) + 7 * ntr)
    if kind == "copies":  # one field of drops in every tracer, shifted by a cell or two
        n = max(2, nx * ny * nz // 900)
        centres = rng.uniform(3 * n).reshape(n, 3) * np.array([nx, ny, nz])
        one = synth.fill_spheres(shape, 1, centres, np.minimum(2.0 + 2.5 * rng.uniform(n), 0.45 * min(shape) - 0.5), np.zeros(n, dtype=int))
        c = np.concatenate([np.roll(one, (0, t // 2, t), (1, 2, 3)) for t in range(ntr)])
    else:  # drops around a few points, one inside the other, and some a little apart
        n = 4 * ntr
        centres = np.repeat(rng.uniform(12).reshape(4, 3), ntr, 0) * np.array([nx, ny, nz]) + 2.5 * (rng.uniform(3 * n).reshape(n, 3) - 0.5)
        radii = np.minimum(1.2 + 4.0 * rng.uniform(n), 0.45 * min(shape) - 0.5)
        centres[::3] += np.array([radii.max() + 2.0, 1.0, 0.0])
        c = synth.fill_spheres(shape, ntr, centres, radii, np.arange(n) % ntr)
    return np.minimum(c, 1.0)


@pytest.mark.parametrize("gap", [0.0, 0.9, 1.5, 2.2, 3.9, 4.3, None])
@pytest.mark.parametrize("kind,shape,ntr", [("copies", (17, 18, 70), 4), ("copies", (24, 20, 64), 2), ("nested", (19, 24, 33), 5),
                                            ("nested", (40, 30, 131), 3), ("nested", (12, 9, 20), 9), ("copies", (4, 30, 40), 3),
                                            ("nested", (30, 30, 4), 3)])
def test_overlapping_drops(ctx, kind, shape, ntr, gap):
    """gap None: the 5x5x5 stencil criterion."""
    import torch

    c = _fields(kind, shape, ntr)
    lab, nd = zip(*[oracle.label(f) for f in c])
    labels = np.stack(lab)
    assert ((labels > 0).sum(0) > 1).any()
    more = 40
    note(f"overlapping drops {kind} {shape} ntr={ntr} gap={gap}")
    full = np.concatenate([c, np.zeros((more,) + shape)])
    args = (full, labels, list(nd), ntr, ntr + more)
    o, ontr, onewt, omoved, rc = oracle.recolor_stencil(*args) if gap is None else oracle.recolor(*args, gap)
    assert rc == 0
    tc = torch.from_numpy(full).to("cuda:0")
    newt = torch.zeros(max(sum(nd), 1), dtype=torch.int32, device="cuda:0")
    args = (tc, ntr, torch.from_numpy(labels).to("cuda:0"), np.array(nd, dtype=np.int32))
    gntr, gmoved = ctx.recolor_tracers_stencil(*args, newt) if gap is None else ctx.recolor_tracers(*args, gap, newt)
    assert (gntr, gmoved) == (ontr, omoved)
    assert np.array_equal(newt.cpu().numpy()[:sum(nd)], onewt)
    assert np.array_equal(tc.cpu().numpy(), o)
