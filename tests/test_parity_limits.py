"""GPU parity on both sides of the limits at which a call takes other kernels or
another turn, where other tests have only one side.

Network forward without records: a workgroup per 64 samples up to 7680 tiles, whole
tiles per wavefront above; with records up to 8192. Outputs are bit-identical.

Reassignment: more neighbours than the list of 32 per drop holds, so that it is
made larger and filled again; the second call in a context finds it large enough.
Bit-exact to the oracle.

Labelling: union tiles of 2048 segments above 1024 of them where a row's words divide
2048, on rows and planes that fill no tile. Exact."""
import numpy as np
import pytest

import oracle
from gpu_util import note, require_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture()
def ctx():
    require_gpu()
    from paper_2407_07463_amd import vofmt

    c = vofmt.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("m", [64 * 7680, 64 * 7680 + 1])
def test_forward_without_records(ctx, m):
    import torch

    from paper_2407_07463_amd import training

    note(f"forward m={m}")
    x = torch.from_numpy(np.random.default_rng(6).random((m, 27), dtype=np.float32)).to("cuda:0")
    params = torch.from_numpy(training.init_params(4)).to("cuda:0")
    plain, recorded = torch.full((m + 1,), 7.0, device="cuda:0"), torch.full((m + 1,), 7.0, device="cuda:0")
    acts = torch.zeros((m, 384), dtype=torch.int16, device="cuda:0")
    ctx.mlp_forward(params, x, plain[:m])
    ctx.mlp_forward(params, x, recorded[:m], acts)
    assert torch.equal(plain, recorded) and float(plain[m]) == 7.0


@pytest.mark.parametrize("gap,neighbours", [(3.2, 32), (3.5, 56), (4.3, 80)])
def test_many_neighbours(ctx, gap, neighbours):
    """Cells two apart in every direction, each a drop; gap 4.3 by the list of boundary cells."""
    import torch

    shape, ntr, more = (12, 18, 24), 2, 62
    full = np.zeros((ntr + more,) + shape)
    full[0, ::2, ::2, ::4] = 1.0
    full[1, ::2, ::2, 2::4] = 0.5
    lab, nd = zip(*[oracle.label(f) for f in full[:ntr]])
    labels = np.stack(lab)
    D = sum(nd)
    assert D == 6 * 9 * 12
    o, ontr, onewt, omoved, rc = oracle.recolor(full, labels, list(nd), ntr, ntr + more, gap)
    assert rc == 0 and omoved > 0
    k = np.stack(np.meshgrid(*[np.arange(-3, 4)] * 3)).reshape(3, -1)
    assert ((4 * (k**2).sum(0) < (1 + gap) ** 2).sum() - 1) == neighbours
    for call in range(2):
        note(f"many neighbours gap={gap} call {call}")
        tc = torch.from_numpy(full).to("cuda:0")
        newt = torch.zeros(D, dtype=torch.int32, device="cuda:0")
        got = ctx.recolor_tracers(tc, ntr, torch.from_numpy(labels).to("cuda:0"), np.array(nd, dtype=np.int32), gap, newt)
        assert got == (ontr, omoved)
        assert np.array_equal(newt.cpu().numpy(), onewt)
        assert np.array_equal(tc.cpu().numpy(), o)


def test_large_union_tiles(ctx):
    """361 tiles of 32 x 32 rows of 2 words a field, the last ones in y and z cut."""
    import torch

    shape, ntr = (601, 599, 70), 3
    rng = np.random.default_rng(8)
    c = np.where(rng.random((ntr,) + shape, dtype=np.float32) < 0.32, 0.5, 0.0)
    note(f"large union tiles {shape} x {ntr}")
    lab = torch.full(c.shape, -7, dtype=torch.int32, device="cuda:0")
    nd = ctx.label_drops(torch.from_numpy(c).to("cuda:0"), lab)
    for t in range(ntr):
        want, k = oracle.label(c[t])
        assert nd[t] == k
        assert np.array_equal(lab[t].cpu().numpy(), want)
