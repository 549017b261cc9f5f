"""GPU parity against the CPU oracle where the split of the work changes with
sizes.

Advection: the marching chunk falls from 32 to 16, 8 and 4 with the number of
wavefronts of a sweep, the initial scan's span with the number of tracer-cells,
and the tracers form groups of even sizes. Bar: 1e-12, the volume-fraction
tolerance of the other advection tests (one or two steps of fields whose
values are O(1)). Rows that are no multiple of 64 cells take lanes across rows,
and words of whole planes (a batch all its boxes): planes below, at and above one
wavefront's and one workgroup's cells, lanes of several rows, in each order of
the sweeps, alone and in a batch with a box whose rows fill their segments. The
flux pass takes 4 list regions as one: mixed cells in one region only (the
first, the last), in every other, and all cells of all regions.

Reassignment: pairs found in LDS tiles of 64 x 8 x 8 cells (reach up to 2, up
to 4; cells that reach no drop but their own left out) or from the list of boundary cells (above, or an axis no longer than the
tile's halo), rows read in groups of 4 cells or one by one, row segments whose
neighbours come by shifts or bit by bit (nx % 64 == 1, nx < 3). Bit-exact.

Interface-cell list: fields of 1 to a few blocks of 8192 cells around the edges
of words, wavefronts and blocks, at addresses that are multiples of 8 bytes (1
for the status) only, and above 4096 blocks, where the counts are scanned. Exact.

Network forward: a workgroup per 64 samples up to 8192 tiles, whole tiles per
wavefront above: the same operations in the same order, so a batch equals its
samples' part of a larger one bit for bit. In training the activation records equal the forward pass's bit for bit
(the same operations in the same order), the loss the mean of its terms to the
rounding of an FP32 sum over m (m 2^-23 relative: all terms are positive).

Labelling: labels written 4, 2 or 1 cells a lane, as rows and the array's
alignment go, union tiles of 512 or 2048 segments, the roots before a workgroup
summed or (above 4096 workgroups) scanned. Exact.

Drop scan: tiles of 128 x 16 x 16 or (few tiles) 128 x 8 x 8 cells, rows of one cell to several segments,
runs that end at a segment's end, more runs than a wavefront notes at once, more
drops in a tile than its table holds. Volumes and centroids within the bounds of
the other moment tests (1e-12 relative; 1e-12 of the box).

Surface-tension force: every group size, one and two groups, and 2 to 32 planes
per workgroup with a remainder. Bit-exact."""
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


@pytest.mark.parametrize("step0", [0, 1, 2])
@pytest.mark.parametrize("shape,ntr", [((1, 1, 1), 1), ((3, 5, 2), 2), ((7, 9, 7), 3), ((4, 2, 65), 5), ((16, 17, 16), 1),
                                       ((15, 8, 127), 4), ((33, 34, 129), 2), ((2, 37, 193), 7)])
def test_lanes_across_rows(ctx, shape, ntr, step0):
    import torch

    boxes = [_random(shape, ntr, 53 + sum(shape)), _random((3, 6, 64), 2, 59)]
    refs = [oracle.advect(c, *s, step0, 2) for c, s in boxes]
    note(f"advect lanes across rows {shape} ntr={ntr} step0={step0}")
    dev = [[torch.from_numpy(a).to("cuda:0") for a in (c, *s)] for c, s in boxes]
    alone = dev[0][0].clone()
    ctx.advect(alone, *dev[0][1:], step0=step0, nsteps=2)
    ctx.advect_batched([tuple(d) for d in dev], step0=step0, nsteps=2)
    torch.cuda.synchronize()
    assert torch.equal(alone, dev[0][0])
    for d, ref in zip(dev, refs):
        assert np.abs(d[0].cpu().numpy() - ref).max() <= TOL


@pytest.mark.parametrize("where", ["first", "last", "alternate", "all"])
def test_list_regions(ctx, where):
    import torch

    shape, ntr = (23, 30, 65), 2  # 90 000 cells: many regions, the last one short
    c, s = _random(shape, ntr, 71)
    flat = c.reshape(-1)
    n = np.arange(flat.size)
    keep = dict(first=n < 300, last=n >= flat.size - 300, alternate=n // 1024 % 2 == 1, all=n >= 0)[where]
    flat[:] = np.where(keep, np.where(flat * (1 - flat) > 0, flat, 0.37), np.round(flat))
    note(f"advect list regions {where}")
    dev = [torch.from_numpy(a).to("cuda:0") for a in (c, *s)]
    alone = dev[0].clone()
    ctx.advect(alone, *dev[1:], step0=0, nsteps=1)
    ctx.advect_batched([tuple(dev)], step0=0, nsteps=1)
    torch.cuda.synchronize()
    assert torch.equal(alone, dev[0])
    assert np.abs(alone.cpu().numpy() - oracle.advect(c, *s, 0, 1)).max() <= TOL


def _labelled(shape, ntr, seed, spread):
    """Small drops, some of them touching or overlapping drops of other tracers, and their labels."""
    nz, ny, nx = shape
    rng = synth.Splitmix64(seed)
    n = max(2 * ntr, nx * ny * nz // 260)
    centres = rng.uniform(3 * n).reshape(n, 3) * np.array([nx, ny, nz])
    radii = np.minimum(1.0 + spread * rng.uniform(n), 0.45 * min(shape) - 0.5).clip(0.4)
    c = synth.fill_spheres(shape, ntr, centres, radii, np.arange(n) % ntr)
    np.minimum(c, 1.0, out=c)
    lab, nd = zip(*[oracle.label(c[t]) for t in range(ntr)])
    return c, np.stack(lab), list(nd)


@pytest.mark.parametrize("gap", [0.0, 0.9, 1.5, 2.2, 3.9, 4.3, None])
@pytest.mark.parametrize("shape,ntr", [((9, 10, 68), 3), ((17, 9, 65), 2), ((8, 8, 64), 5), ((7, 25, 131), 4),
                                       ((5, 5, 6), 2), ((4, 9, 20), 2), ((3, 6, 2), 1), ((16, 8, 256), 3)])
def test_reassignment_tiles(ctx, shape, ntr, gap):
    """gap None: the 5x5x5 stencil criterion."""
    import torch

    c, labels, nd = _labelled(shape, ntr, 900 + sum(shape), 1.6)
    maxt = ntr + 24
    note(f"reassignment tiles {shape} ntr={ntr} gap={gap}")
    full = np.concatenate([c, np.zeros((24,) + shape)])
    if gap is None:
        o, ontr, onewt, omoved, rc = oracle.recolor_stencil(full, labels, nd, ntr, maxt)
    else:
        o, ontr, onewt, omoved, rc = oracle.recolor(full, labels, nd, ntr, maxt, gap)
    assert rc == 0
    tc = torch.from_numpy(full).to("cuda:0")
    lab = torch.from_numpy(np.ascontiguousarray(labels)).to("cuda:0")
    newt = torch.zeros(max(sum(nd), 1), dtype=torch.int32, device="cuda:0")
    args = (tc, ntr, lab, np.array(nd, dtype=np.int32))
    gntr, gmoved = ctx.recolor_tracers_stencil(*args, newt) if gap is None else ctx.recolor_tracers(*args, gap, newt)
    assert (gntr, gmoved) == (ontr, omoved)
    assert np.array_equal(newt.cpu().numpy()[:sum(nd)], onewt)
    assert np.array_equal(tc.cpu().numpy(), o)


@pytest.mark.parametrize("shape,ntr", [((3, 17, 70), 5), ((33, 9, 65), 6), ((7, 8, 129), 7), ((5, 20, 64), 10),
                                       ((2, 3, 5), 15), ((1, 1, 1), 3), ((561, 120, 65), 1), ((1101, 120, 65), 2)])
def test_force_groups(ctx, shape, ntr):
    import torch

    rng = np.random.default_rng(sum(shape) + ntr)
    c = rng.random((ntr,) + shape)
    c[c < 0.4] = 0.0
    kappa = rng.standard_normal((ntr,) + shape)
    kappa[rng.random((ntr,) + shape) < 0.5] = np.nan
    note(f"force {shape} ntr={ntr}")
    f = [torch.empty(shape, dtype=torch.float64, device="cuda:0") for _ in range(3)]
    ctx.csf_force(torch.from_numpy(c).to("cuda:0"), torch.from_numpy(kappa).to("cuda:0"), 0.7, *f)
    for g, o in zip(f, oracle.csf_force(c, kappa, 0.7)):
        assert np.array_equal(g.cpu().numpy(), o)


@pytest.mark.parametrize("shape", [(1, 1, 1), (1, 1, 63), (1, 5, 13), (1, 1, 2047), (3, 683, 1), (1, 1, 2049), (8191, 1, 1),
                                   (1, 8193, 1), (25, 33, 31), (1, 127, 129), (323, 322, 324)])
def test_interface_list(ctx, shape):
    import torch

    n = int(np.prod(shape))
    rng = np.random.default_rng(n)
    c = np.zeros((2, n + 1))  # the second field is only 8-byte aligned for odd n + 1
    hit = rng.random(n) < 0.03
    c[1, :n][hit] = rng.random(int(hit.sum()))
    c[1, :n][~hit & (rng.random(n) < 0.5)] = 1.0
    field = c[1, :n].reshape(shape)
    want = np.flatnonzero((field.ravel() > 1e-12) & (field.ravel() < 1 - 1e-12))
    note(f"interface list {shape}")
    dev = "cuda:0"
    f = torch.from_numpy(c).to(dev)[1, :n].reshape(shape)
    m = len(want)
    xs = torch.zeros((m + 1, 27), dtype=torch.float32, device=dev)
    cell, sign = torch.zeros(m + 1, dtype=torch.int32, device=dev), torch.zeros(m + 1, dtype=torch.int8, device=dev)
    assert ctx.mlp_stencils(f, xs, cell, sign) == m
    assert np.array_equal(cell.cpu().numpy()[:m], want)
    kappa = torch.zeros(2 * n + 1, dtype=torch.float64, device=dev)[n + 1:].reshape(shape)
    status = torch.full((2 * n + 1,), 77, dtype=torch.uint8, device=dev)
    ctx.curvature_hf(f, kappa, status[n:2 * n].reshape(shape))
    st = status.cpu().numpy()
    assert np.array_equal(np.flatnonzero(st[n:2 * n]), want)
    assert np.all(st[:n] == 77) and st[2 * n] == 77  # nothing written beside the field
    assert np.isnan(kappa.cpu().numpy().ravel()[st[n:2 * n] == 0]).all()


def _separate(kind, shape, rng):
    """One field of drops that nowhere touch and span less than half of every axis."""
    nz, ny, nx = shape
    k, j, i = np.meshgrid(*[np.arange(n) for n in shape], indexing="ij")
    inside = (k < nz - nz % 2) & (j < ny - ny % 2) & (i < nx - 1)  # (no contact across the boundary)
    if kind == "cells":  # single cells in a checkered pattern
        hit = ((k + j + i) % 2 == 0) & (i < nx - nx % 2) & (rng.random(shape) < 0.5)
    elif kind == "bars":  # runs of cells of 1 to 3 n/8 along x, in every other row and plane
        cut = rng.random((nz, ny, 1)) * nx
        length = max(1, 3 * nx // 8)
        hit = (k % 2 == 0) & (j % 2 == 0) & ((i + cut.astype(int)) % (length + 1) != 0) & (rng.random((nz, ny, 1)) < 0.8)
    else:  # blocks of up to 5 x 4 x 6 cells
        hit = (k % 6 < 5) & (j % 5 < 4) & (i % 7 < 6) & (rng.random(shape) < 0.97) & (k < nz - nz % 6) & (j < ny - ny % 5) \
            & (i < nx - nx % 7)
    return np.where(hit & inside, 0.1 + 0.9 * rng.random(shape), 0.0)


@pytest.mark.parametrize("kind,shape", [("blocks", (17, 16, 128)), ("blocks", (16, 17, 129)), ("blocks", (36, 35, 300)),
                                        ("bars", (33, 5, 65)), ("bars", (4, 40, 63)), ("bars", (18, 20, 300)),
                                        ("bars", (2, 3, 1000)), ("cells", (16, 16, 128)), ("cells", (5, 6, 200)),
                                        ("cells", (40, 3, 3))])
def test_drop_scan_tiles(ctx, kind, shape):
    _check_drop_scan(ctx, kind, shape)


@pytest.mark.parametrize("kind,shape", [("cells", (736, 721, 5)), ("bars", (1441, 368, 5)), ("bars", (512, 1024, 5))])
def test_drop_scan_tile_sizes(ctx, kind, shape):
    """More than 4096 tiles of 16 rows by 16 planes, and 4096."""
    _check_drop_scan(ctx, kind, shape)


def _check_drop_scan(ctx, kind, shape):
    import torch

    nz, ny, nx = shape
    rng = np.random.default_rng(sum(shape))
    c = np.stack([_separate(kind, shape, rng) for _ in range(2)])
    lab, nd = zip(*[oracle.label(f) for f in c])
    D = sum(nd)
    note(f"drop scan {kind} {shape} drops={D}")
    dev = "cuda:0"
    vol, xyz = torch.zeros(D, dtype=torch.float64, device=dev), torch.zeros((D, 3), dtype=torch.float64, device=dev)
    ref = [oracle.drop_moments(c[t], lab[t], nd[t]) for t in range(2)]
    assert all(r[2] == 0 for r in ref)
    ctx.drop_moments(torch.from_numpy(c).to(dev), torch.from_numpy(np.stack(lab)).to(dev), np.array(nd, dtype=np.int32), vol, xyz)
    rv, rx = np.concatenate([r[0] for r in ref]), np.concatenate([r[1] for r in ref])
    assert np.all(np.abs(vol.cpu().numpy() - rv) <= 1e-12 * rv)
    box = np.array([nx, ny, nz], dtype=np.float64)
    d = np.abs(xyz.cpu().numpy() - rx)
    assert np.all(np.minimum(d, box - d) <= 1e-12 * box)


@pytest.fixture(scope="module")
def large_forward(ctx):
    import torch

    from paper_2407_07463_amd import training

    m = 64 * 8192 + 17
    x = torch.from_numpy(np.random.default_rng(5).random((m, 27), dtype=np.float32)).to("cuda:0")
    params = torch.from_numpy(training.init_params(4)).to("cuda:0")
    y = torch.empty(m, dtype=torch.float32, device="cuda:0")
    acts = torch.zeros((m, 384), dtype=torch.int16, device="cuda:0")
    ctx.mlp_forward(params, x, y, acts)
    return params, x, y, acts


@pytest.mark.parametrize("m,first", [(1, 0), (16, 3), (63, 64), (65, 1000), (4096, 5), (64 * 8192, 17)])
@pytest.mark.parametrize("records", [False, True])
def test_forward_tiles(ctx, large_forward, m, first, records):
    import torch

    params, x, y_all, acts_all = large_forward
    note(f"forward m={m} first={first} records={records}")
    y = torch.full((m + 1,), 7.0, dtype=torch.float32, device="cuda:0")
    acts = torch.full((m + 1, 384), 7, dtype=torch.int16, device="cuda:0") if records else None
    ctx.mlp_forward(params, x[first:first + m].contiguous(), y[:m], None if acts is None else acts[:m])
    assert torch.equal(y[:m], y_all[first:first + m]) and float(y[m]) == 7.0
    if records:
        assert torch.equal(acts[:m], acts_all[first:first + m]) and bool((acts[m] == 7).all())


@pytest.mark.parametrize("m", [1, 15, 17, 64, 65, 1000, 65536, 65537])
def test_training_forward_tiles(ctx, m):
    import torch

    from paper_2407_07463_amd import training

    rng = np.random.default_rng(m)
    x = torch.from_numpy(rng.random((m, 27), dtype=np.float32)).to("cuda:0")
    t = torch.from_numpy(rng.standard_normal(m).astype(np.float32)).to("cuda:0")
    params = torch.from_numpy(training.init_params(3)).to("cuda:0")
    y = torch.empty(m, dtype=torch.float32, device="cuda:0")
    acts = torch.zeros((m, 384), dtype=torch.int16, device="cuda:0")
    trace = torch.zeros((m, 640), dtype=torch.int16, device="cuda:0")
    note(f"training forward m={m}")
    ctx.mlp_forward(params, x, y, acts)
    loss = ctx.mlp_train_step(params, torch.zeros_like(params), torch.zeros_like(params), 1, 1e-3, x, t, trace=trace)
    assert torch.equal(trace[:, :384], acts)
    yd, td = y.double(), t.double()
    want = float(((yd - td) ** 2 / td.abs().clamp(min=0.05) ** 2).mean())
    assert abs(loss - want) <= (m + 8) * 2.0**-23 * want


@pytest.mark.parametrize("shape,offset", [((7, 9, 64), 0), ((7, 9, 64), 1), ((7, 9, 64), 2), ((6, 5, 66), 0), ((6, 5, 66), 1),
                                          ((5, 7, 67), 0), ((9, 33, 260), 0), ((3, 1025, 3), 0), ((2100, 2001, 1), 0),
                                          ((300, 290, 65), 0)])
def test_label_forms(ctx, shape, offset):
    """offset: of the label array from a 16-byte boundary, in labels."""
    import torch

    rng = np.random.default_rng(sum(shape) + offset)
    c = np.where(rng.random((2,) + shape) < 0.3, rng.random((2,) + shape), 0.0)
    note(f"labels {shape} offset={offset}")
    buf = torch.full((c.size + offset + 1,), -7, dtype=torch.int32, device="cuda:0")
    lab = buf[offset:offset + c.size].reshape(c.shape)
    nd = ctx.label_drops(torch.from_numpy(c).to("cuda:0"), lab)
    for t in range(2):
        want, k = oracle.label(c[t])
        assert nd[t] == k
        assert np.array_equal(lab[t].cpu().numpy(), want)
    assert int(buf[-1]) == -7 and (offset == 0 or bool((buf[:offset] == -7).all()))
