"""GPU parity of the nearest-pair search where the periodic image matters: points at
exactly half the box from one another, outside the box, at the same place, and box
edges that halve inexactly; one to many slices of candidates. Indices, ties and
histograms bit-exact, moments to 1e-12 of their scale."""
import numpy as np
import pytest

import oracle
from gpu_util import note, require_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["lattice", "outside", "thirds", "same"])
@pytest.mark.parametrize("n", [2, 64, 257, 1000, 5000])
def test_nearest_images(kind, n):
    torch = require_gpu()
    from paper_2407_07463_amd import vofmt

    rng = np.random.default_rng(n)
    box = np.array([24.0, 16.0, 20.0]) if kind != "thirds" else np.array([0.7, 1.0 / 3.0, 5e-3])
    if kind == "lattice":  # distances of half the box in every axis, many ties
        xyz = rng.integers(0, 4, (n, 3)) * (box / 4)
    elif kind == "thirds":
        xyz = rng.random((n, 3)) * box
        xyz[1::2] = (xyz[::2][:len(xyz[1::2])] + box / 2) % box
    else:
        xyz = rng.random((n, 3)) * box
        if kind == "outside":
            xyz += rng.integers(-2, 3, (n, 3)) * box * 0.75
        else:
            xyz[n // 2:] = xyz[:n - n // 2]
    nr, nth = 16, 8
    r2e = (np.arange(nr + 1) * (box.max() / nr)) ** 2
    ce = np.cos(np.arange(nth + 1) * np.pi / nth)
    note(f"nearest images {kind} n={n}")
    want = oracle.nearest_pair_stats(xyz, box, 1, r2e, ce)
    ctx = vofmt.Context(0)
    try:
        z = lambda k, dt: torch.zeros(k, dtype=dt, device="cuda:0")  # noqa: E731
        idx, ties, hist = z(n, torch.int32), z(n, torch.int32), z(nr * nth + 1, torch.int64)
        M, R = z(3, torch.float64), z(9, torch.float64)
        ctx.nearest_pair_stats(torch.from_numpy(xyz).to("cuda:0"), box, 1, r2e, ce, idx, ties, hist, M, R)
    finally:
        ctx.close()
    assert np.array_equal(idx.cpu().numpy(), want["nn_index"])
    assert np.array_equal(ties.cpu().numpy(), want["nn_ties"])
    assert np.array_equal(hist.cpu().numpy().view(np.uint64), want["raw_hist"])
    scale = float(want["R"].trace())
    assert np.abs(M.cpu().numpy() - want["M"]).max() <= 1e-12 * np.sqrt(scale)
    assert np.abs(R.cpu().numpy().reshape(3, 3) - want["R"]).max() <= 1e-12 * scale
