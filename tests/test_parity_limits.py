"""GPU parity on both sides of the limits at which a call takes other kernels or
another turn, where other tests have only one side.

Network forward without records: a workgroup per 64 samples up to 7680 tiles, whole
tiles per wavefront above; with records up to 8192. Outputs are bit-identical."""
import numpy as np
import pytest

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
