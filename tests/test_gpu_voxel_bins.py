"""Voxelization by bin of cells (clouds of at least 524 288 points, or a million where these are over 200 a tile, on grids of at least 1 024
tiles of 65 536 cells) against the oracle, with bins of a quarter of a tile and of a whole one, at the point counts of a bin where its
form changes."""
import numpy as np
import pytest
import torch

import oracle
from helpers import assert_features_close
from paper_2507_04123_amd import binding as B
from paper_2507_04123_amd.configs import SUBM, VoxelSpec
from paper_2507_04123_amd.pipeline import cells_of
from test_gpu_stacks import _kernels_in

pytestmark = pytest.mark.gpu

N = 524288
GRID = (4096, 4096, 16)                # 4 096 tiles of 16 lines (y) each: a quarter, the bins of over 100 points a tile, is 4 lines
WIDE = (4096, 4096, 24)                # 6 144 tiles: bins of a whole one
BINS, POINTS = 7, 6                    # launches


def _cloud(seed, n, fullest, heavy, frames):
    """n points in layers 0 .. 3; of lines 1600 .. 1615 in layer 2 of the last frame the first four hold `fullest` of them, the others
    none."""
    rng = np.random.RandomState(seed)
    p = np.empty((n, 4), np.float32)
    p[:, 0] = rng.randint(0, 4096, n) + 0.25
    p[:, 1] = rng.randint(0, 4096, n) + 0.5
    p[:, 2] = rng.randint(0, 4, n) + 0.75
    p[:, 3] = rng.uniform(0, 1, n)
    b = rng.randint(0, frames, n).astype(np.int32)
    inside = (b == frames - 1) & (p[:, 2] == 2.75) & (p[:, 1] >= 1600) & (p[:, 1] < 1616)
    p[inside, 1] -= 800.0              # that bin is filled on purpose
    t = rng.permutation(n)[:fullest]
    b[t] = frames - 1
    p[t, 2], p[t, 1], p[t, 0] = 2.75, 1600.5 + rng.randint(0, 4, fullest), rng.randint(0, 4096, fullest) + 0.5
    if heavy:                          # voxels of 2 .. 600 points, ends of lines among them
        at = 0
        for k, x in ((2, 0), (3, 4095), (4, 31), (5, 32), (9, 100), (600, 4095)):
            p[t[at:at + k], 0], p[t[at:at + k], 1] = x + 0.5, 1600.5 if x != 4095 else 1603.5
            p[t[at:at + k], 3] = rng.uniform(0, 1, k)
            at += k
    p[rng.permutation(n)[:50], 0] = -1.0                  # dropped
    b[rng.permutation(n)[:50]] = frames                   # dropped
    return p, b


def _launches(ctx, spec, n, cap):
    i32 = dict(dtype=torch.int32, device="cuda")
    pts, out = torch.zeros((n, 4), device="cuda"), [torch.zeros((cap, 4), **i32), torch.zeros((cap, 4), device="cuda"), torch.zeros(cap, **i32)]
    nv = torch.zeros(1, **i32)
    return _kernels_in(lambda: ctx.voxelize(pts, None, spec, cap, *out, nv))


@pytest.mark.parametrize("layers,n,launches", [(2, 524288, POINTS), (4, 524288, POINTS), (4, 737280, POINTS), (16, 524287, POINTS), (16, 524288, BINS),
                                               (16, 819200, BINS), (16, 819201, POINTS), (16, 999999, POINTS), (16, 1000000, BINS),
                                               (6, 1105920, BINS), (6, 1105921, POINTS)])
def test_clouds_that_go_by_bins(layers, n, launches):
    """512 tiles, 1 024 and more; up to 200 points a tile from 524 288 on, over 200 from a million on, over 720 never."""
    grid = (4096, 4096, layers)
    ctx = B.Context(n, 1000, cells_of(grid, 1), n_slots=1)
    assert _launches(ctx, VoxelSpec((0.0, 0.0, 0.0), (1.0, 1.0, 1.0), grid), n, 1000) == launches
    ctx.close()


def _check(ctx, pts, batch, spec, cap, stride=4, lp=torch.float16, launches=BINS, rtol=4e-5):
    n = len(pts)
    assert _launches(ctx, spec, n, cap) == launches
    wide = np.zeros((n, stride), np.float32)
    wide[:, :4] = pts
    i32 = dict(dtype=torch.int32, device="cuda")
    coords, feats, counts = torch.full((cap, 4), -7, **i32), torch.full((cap, 4), 9.0, device="cuda"), torch.full((cap,), 9, **i32)
    lpt = torch.zeros((cap, 4), dtype=lp, device="cuda")
    nv = torch.zeros(1, **i32)
    ctx.voxelize(torch.from_numpy(wide).cuda(), torch.from_numpy(batch).cuda(), spec, cap, coords, feats, counts, nv, feats_lp=lpt)
    oc, om, on = oracle.voxelize(pts, batch, spec.lo, spec.vs, spec.grid, n_batch=spec.n_batch)
    m = min(len(oc), cap)
    assert int(nv.item()) == m
    assert np.array_equal(coords[:m].cpu().numpy(), oc[:m]) and bool((coords[m:] == -7).all())
    assert np.array_equal(counts[:m].cpu().numpy(), on[:m])
    # fp32 sums of up to 600 values of 0 .. 4096 against fp64: 600 * 2^-24 relative to the largest partial sum, over the mean (of 6 100: 4e-4)
    assert_features_close(feats[:m].cpu().numpy(), om[:m], rtol, "means")
    assert torch.equal(lpt[:m], feats[:m].to(lp)) and bool((lpt[m:] == 0).all())
    bound = min(n, cap)
    assert not feats[m:bound].any() and not counts[m:bound].any()
    assert bool((feats[bound:] == 9.0).all()) and bool((counts[bound:] == 9).all())
    if len(oc) <= cap:
        ctx.status_sync()
        # the index left in the slot against one rebuilt from the coordinates
        nbr, ref = torch.zeros((27, cap), **i32), torch.zeros((27, cap), **i32)
        ctx.build_kmap(SUBM, coords, nv, cap, spec.grid, spec.n_batch, cap, nbr, nv, in_slot=0)
        ctx.build_kmap(SUBM, coords, nv, cap, spec.grid, spec.n_batch, cap, ref, nv)
        ctx.status_sync()
        assert torch.equal(nbr[:, :m], ref[:, :m])
    else:
        with pytest.raises(B.Emc2Error) as e:
            ctx.status_sync()
        assert e.value.status == B.ERR_CAPACITY
    return feats, m


# (30 000 points: two chunks of points, four parts of voxels; 200 000: 13 of each)
@pytest.mark.parametrize("grid", [GRID, WIDE])
@pytest.mark.parametrize("fullest,heavy", [(1, False), (3072, True), (3073, True), (30000, True), (200000, True)])
def test_points_of_the_fullest_bin(fullest, heavy, grid):
    spec = VoxelSpec((0.0, 0.0, 0.0), (1.0, 1.0, 1.0), grid)
    ctx = B.Context(N + 1000, N + 1000, cells_of(grid, 1), n_slots=1)
    pts, batch = _cloud(3, N, fullest, heavy, 1)
    a, m = _check(ctx, pts, batch, spec, N + 500)
    # another cloud into the same slot: lines that only the first one filled hold nothing any more
    pts2, batch2 = _cloud(4, N, 777, heavy, 1)
    _check(ctx, pts2, batch2, spec, N + 500, stride=5, lp=torch.bfloat16)
    if not heavy:                      # voxels of up to four points: the same bits for any order of the points
        o = np.random.RandomState(1).permutation(N)
        b, _ = _check(ctx, pts[o], batch[o], spec, N + 500)
        assert torch.equal(a[:m], b[:m])
    ctx.close()


@pytest.mark.parametrize("layers,shift", [(16, 14), (80, 16)])
def test_more_large_bins_than_blocks(layers, shift):
    """More bins of over 3 072 points than the 512 blocks that mark their cells and the 256 blocks that take their parts: each block takes
    a second one, of another number of voxels.  Bins of a quarter of a tile (16 layers: 4 096 tiles) and of a whole one (80 layers:
    20 480, under 100 points each)."""
    grid, large, n = (4096, 4096, layers), 600, 1950000
    rng = np.random.RandomState(shift)
    n_bins = 4096 * 4096 * layers >> shift
    assert n >= 100 * 256 * layers if shift == 14 else n < 100 * 256 * layers
    bins = rng.permutation(n_bins)[:large].astype(np.int64)
    points = 3073 + rng.randint(0, 80, large)
    span = np.array([16, 127, 128, 129, 1000, 1 << 13, 1 << shift])[np.arange(large) % 7]        # cells that its points are drawn from
    key = np.concatenate([np.repeat(bins << shift, points) + rng.randint(0, 1 << 30, points.sum()) % np.repeat(span, points),
                          rng.randint(0, n_bins << shift, n - points.sum())])
    key = key[rng.permutation(n)]
    p = np.empty((n, 4), np.float32)
    p[:, 0], p[:, 1], p[:, 2], p[:, 3] = key % 4096 + 0.5, key // 4096 % 4096 + 0.25, key // 4096 ** 2 + 0.75, rng.uniform(0, 1, n)
    ctx = B.Context(n, n, cells_of(grid, 1), n_slots=1)
    _check(ctx, p, np.zeros(n, np.int32), VoxelSpec((0.0, 0.0, 0.0), (1.0, 1.0, 1.0), grid), n)
    ctx.close()


@pytest.mark.parametrize("grid", [GRID, WIDE])
def test_most_points_in_one_bin(grid):
    """A bin with 16 384 voxels, its parts of the most that a block can hold; then 300 000 points in 50 of them: more parts than that
    take a voxel, and voxels of 6 000 points."""
    spec = VoxelSpec((0.0, 0.0, 0.0), (1.0, 1.0, 1.0), grid)
    ctx = B.Context(N, N, cells_of(grid, 1), n_slots=1)
    for n, voxels in ((60000, 16384), (300000, 50)):
        pts, batch = _cloud(9, N, 1, False, 1)
        at, cell = np.random.RandomState(2).permutation(N)[:n], np.arange(n) % voxels
        pts[at, 0], pts[at, 1], pts[at, 2] = cell % 4096 + 0.5, 1600.5 + cell // 4096, 2.75
        _check(ctx, pts, batch, spec, N, rtol=4e-4)
    ctx.close()


def test_points_of_all_frames_mixed_and_capacity():
    """Bins of a tile; frames in any order: a block's points lie in more bins than it counts in LDS at a time.  Then a capacity below the voxels, and a cloud of
    one point less than the limit, which takes the pass over single points, into the same slot."""
    grid = (4096, 4096, 4)
    spec = VoxelSpec((0.0, 0.0, 0.0), (1.0, 1.0, 1.0), grid, n_batch=9)
    ctx = B.Context(N + 77, N + 77, cells_of(grid, 9), n_slots=1)
    pts, batch = _cloud(5, N + 77, 5000, True, 9)
    _check(ctx, pts, batch, spec, N + 77)
    _check(ctx, pts, batch, spec, 100001)
    _check(ctx, pts[: N - 1], batch[: N - 1], spec, N, launches=POINTS)
    _check(ctx, pts, batch, spec, N + 77)
    ctx.close()


def test_captured_voxelization_by_bin_replays():
    """Recorded once, replayed on other points, with eager work between the replays."""
    spec = VoxelSpec((0.0, 0.0, 0.0), (1.0, 1.0, 1.0), GRID)
    ctx = B.Context(N, N, cells_of(GRID, 1), n_slots=1)
    i32 = dict(dtype=torch.int32, device="cuda")
    coords, feats, counts, nv = torch.zeros((N, 4), **i32), torch.zeros((N, 4), device="cuda"), torch.zeros(N, **i32), torch.zeros(1, **i32)
    clouds = [torch.from_numpy(_cloud(s, N, f, False, 1)[0]).cuda() for s, f in ((6, 3000), (7, 20000), (8, 10))]
    pts = clouds[0].clone()
    run = lambda: ctx.voxelize(pts, None, spec, N, coords, feats, counts, nv)
    run()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        run()
    for c in clouds + clouds[:1]:
        pts.copy_(c)
        run()
        torch.cuda.synchronize()
        exp = [t.clone() for t in (coords, feats, counts, nv)]
        for t in (coords, feats, counts, nv):
            t.fill_(-3)
        g.replay()
        torch.cuda.synchronize()
        m = int(exp[3].item())
        assert int(nv.item()) == m
        few = exp[2][:m] <= 4           # the sum of more points has no order of its own
        assert torch.equal(coords[:m], exp[0][:m]) and torch.equal(counts[:m], exp[2][:m])
        assert torch.equal(feats[:m][few], exp[1][:m][few]) and torch.allclose(feats[:m], exp[1][:m], rtol=1e-5)
    ctx.close()
