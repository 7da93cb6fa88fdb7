"""Indexes built from marks: a slot that held another index before, marks that the calls of a context share, sites by the word."""
import numpy as np
import pytest
import torch

import oracle
from helpers import assert_features_close
from paper_2507_04123_amd import binding as B
from paper_2507_04123_amd.configs import F16, VoxelSpec
from paper_2507_04123_amd.pipeline import cells_of
from test_gpu_stacks import _Bufs, _kernels_in, _same

pytestmark = pytest.mark.gpu


def _voxels(ctx, keys, grid, cap):
    """The sites `keys` of `grid` through the voxelizer, and the submanifold map made from the slot's index."""
    gx, gy, _ = grid
    k = np.asarray(keys, np.int64)
    pts = np.stack([k % gx + 0.5, k // gx % gy + 0.5, k // (gx * gy) + 0.5, np.ones(len(k))], axis=1).astype(np.float32)
    i32 = dict(dtype=torch.int32, device="cuda")
    coords, feats, counts = torch.zeros((cap, 4), **i32), torch.zeros((cap, 4), device="cuda"), torch.zeros(cap, **i32)
    n, nbr = torch.zeros(1, **i32), torch.full((27, cap), -5, **i32)
    spec = VoxelSpec((0.0, 0.0, 0.0), (1.0, 1.0, 1.0), grid)
    ctx.voxelize(torch.from_numpy(pts).cuda(), None, spec, cap, coords, feats, counts, n, index_slot=0)
    ctx.build_kmap(B.SUBM, coords, n, cap, grid, 1, cap, nbr, n, in_slot=0)
    ctx.status_sync()
    m = int(n.item())
    return coords[:m].clone(), nbr[:, :m].clone()


def _expected(keys, grid):
    gx, gy, gz = grid
    keys = np.unique(np.asarray(keys, np.int64))
    z, y, x = keys // (gx * gy), keys // gx % gy, keys % gx
    nbr = np.full((27, len(keys)), -1, np.int64)
    for t in range(27):
        zz, yy, xx = z + t // 9 - 1, y + t // 3 % 3 - 1, x + t % 3 - 1
        ok = (zz >= 0) & (zz < gz) & (yy >= 0) & (yy < gy) & (xx >= 0) & (xx < gx)
        want = (zz * gy + yy) * gx + xx
        at = np.minimum(np.searchsorted(keys, want), len(keys) - 1)
        hit = ok & (keys[at] == want)
        nbr[t, hit] = at[hit]
    return np.stack([0 * z, z, y, x], axis=1), nbr


# 8 192 words of the index, the most that one block takes; a word more; many tiles
@pytest.mark.parametrize("grid", [(32, 128, 64), (32, 8193, 1), (200, 201, 41)])
def test_slot_that_held_another_index(grid):
    cells, small = int(np.prod(grid)), (20, 10, 3)
    rng = np.random.RandomState(cells)
    cap = 20000
    ctx = B.Context(cap, cap, cells_of(grid, 1), n_slots=1)
    many, line = rng.randint(0, cells, 15000), np.arange(cells - 700, cells)
    for keys, g in ((many, grid), (line, grid), (np.arange(100), small), ([0, cells - 1], grid), (many[:40], grid), (many, grid)):
        coords, nbr = _voxels(ctx, keys, g, cap)
        want_c, want_n = _expected(keys, g)
        assert np.array_equal(coords.cpu().numpy(), want_c) and np.array_equal(nbr.cpu().numpy(), want_n)
    ctx.close()


def _sites(ctx, how, keys, grid, slot=0):
    """The sites `keys` of a grid of 32 cells a row (a word of the index is a row of y) left in `slot` by one of the three calls that build from
    marks."""
    rows, keys = grid[1], np.asarray(keys, np.int64)
    cap = max(len(keys), 1)
    i32 = dict(dtype=torch.int32, device="cuda")
    coords, counts, n = torch.zeros((cap, 4), **i32), torch.zeros(cap, **i32), torch.zeros(1, **i32)
    spec = VoxelSpec((0.0, 0.0, 0.0), (1.0, 1.0, 1.0), grid)
    if how == "voxelize":
        pts = np.full((cap, 4), -1.0, np.float32)                            # (without a site: a point outside)
        pts[:len(keys), 0], pts[:len(keys), 1], pts[:len(keys), 2] = keys % 32 + 0.5, keys // 32 + 0.5, 0.5
        ctx.voxelize(torch.from_numpy(pts).cuda(), None, spec, cap, coords, torch.zeros((cap, 4), device="cuda"), counts, n, index_slot=slot)
    elif how == "pool":
        depth = np.zeros((rows, 32), np.float32)                             # pixel (y, x) at depth 1 is cell (0, y, x)
        depth.flat[keys] = 1.0
        q = [1, 0, 0, 0.5, 0, 1, 0, 0.5, 0, 0, 0, 0.5]
        img = torch.zeros((rows, 32, 8), dtype=torch.float16, device="cuda")
        ctx.pool_image(img, torch.from_numpy(depth).cuda(), q, spec, B.POOL_MAX, cap, coords,
                       torch.zeros((cap, 8), dtype=torch.float16, device="cuda"), counts, n, index_slot=slot)
    else:
        at = torch.zeros((cap, 4), **i32)
        at[:len(keys)] = torch.from_numpy(np.stack([0 * keys, 0 * keys, keys // 32, keys % 32], axis=1).astype(np.int32)).cuda()
        f, m, none = torch.zeros((cap, 8), dtype=torch.float16, device="cuda"), torch.full((1,), len(keys), **i32), torch.zeros(1, **i32)
        ctx.fuse(F16, at, f, m, cap, at, f, none, cap, grid, 1, cap, coords, torch.zeros((cap, 16), dtype=torch.float16, device="cuda"), n,
                 out_slot=slot)
    ctx.status_sync()
    assert int(n.item()) == len(keys)
    return coords, n, cap


def _line_and_around(words):
    """Cells of the last line (16 words) of a grid of `words` words, and the cells of the words before and behind it."""
    first = (words - 1) // 16 * 16
    around = [w for w in (first - 1, *range(first + 16, first + 56)) if w >= 0]
    return np.arange(first * 32, (first + 16) * 32), np.concatenate([np.arange(w * 32, w * 32 + 32) for w in around])


def _small_sites(words, held):
    return ([5] if words > 16 else []) + ([(words - 1) * 32 + 31] if held else [])


# The last line of a smaller grid, full of an older index's sites: words of both its halves, of one, all of them are the grid's.  The line
# holds a new site or none.  What the next larger grid finds in the line, through a map, a stride-2 level and a stack in the slot.
@pytest.mark.parametrize("held", [False, True])
@pytest.mark.parametrize("words", [1, 8, 9, 15, 16, 19, 24, 25, 8104])
@pytest.mark.parametrize("rows", [8192, 8200])                                # in one block; in tiles
@pytest.mark.parametrize("how", ["voxelize", "pool", "fuse"])
def test_last_line_of_a_smaller_grid(how, rows, words, held):
    large, small = (32, rows, 1), (32, words, 1)
    line, around = _line_and_around(words)
    ctx = B.Context(rows * 32, 8192, rows * 32, n_slots=1)
    _sites(ctx, how, np.sort(np.concatenate([line, around])), large)
    _sites(ctx, how, _small_sites(words, held), small)
    coords, n, cap = _sites(ctx, how, around, large)
    nbr = torch.full((27, cap), -5, dtype=torch.int32, device="cuda")
    ctx.build_kmap(B.SUBM, coords, n, cap, large, 1, cap, nbr, n, in_slot=0)
    ctx.status_sync()
    want_c, want_n = _expected(around, large)
    assert np.array_equal(coords.cpu().numpy(), want_c) and np.array_equal(nbr.cpu().numpy(), want_n)
    ctx.close()


@pytest.mark.parametrize("words", [8, 19, 25])
def test_last_line_of_a_smaller_grid_then_a_strided_level(words):
    fine, coarse = (64, 16384, 1), (32, 8192, 1)                              # 8 192 words: counted by one block, which asks no flags
    line, around = _line_and_around(words)
    got = []
    for used in (True, False):
        ctx = B.Context(8192 * 32, 8192, 64 * 16384, n_slots=2)
        if used:
            _sites(ctx, "voxelize", np.sort(np.concatenate([line, around])), coarse)
            _sites(ctx, "voxelize", _small_sites(words, False), (32, words, 1))
        pts = np.stack([2 * (around % 32) + 0.5, 2 * (around // 32) + 0.5, 0 * around + 0.5, 0 * around], axis=1).astype(np.float32)
        cap = len(around)
        i32 = dict(dtype=torch.int32, device="cuda")
        c0, f0, k0, n0 = torch.zeros((cap, 4), **i32), torch.zeros((cap, 4), device="cuda"), torch.zeros(cap, **i32), torch.zeros(1, **i32)
        ctx.voxelize(torch.from_numpy(pts).cuda(), None, VoxelSpec((0.0, 0.0, 0.0), (1.0, 1.0, 1.0), fine), cap, c0, f0, k0, n0, index_slot=1)
        big = 4096
        c1, n1, nbr = torch.zeros((big, 4), **i32), torch.zeros(1, **i32), torch.full((27, big), -5, **i32)
        ctx.build_kmap(B.STRIDED, c0, n0, cap, fine, 1, big, nbr, n1, out_coords=c1, in_slot=1, out_slot=0)
        ctx.status_sync()
        m = int(n1.item())
        got.append((m, c1[:m].cpu().numpy(), nbr[:, :m].cpu().numpy()))
        ctx.close()
    assert got[0][0] == got[1][0] == len(around)
    assert np.array_equal(got[0][1], got[1][1]) and np.array_equal(got[0][2], got[1][2])


@pytest.mark.parametrize("words", [8, 19, 25])
@pytest.mark.parametrize("rows", [8192, 8200])                                # the stack in one launch; in several
def test_last_line_of_a_smaller_grid_then_a_stack(rows, words):
    large = (32, rows, 1)
    line, around = _line_and_around(words)
    spec = VoxelSpec((0.0, 0.0, 0.0), (1.0, 1.0, 1.0), large)
    pts = np.stack([around % 32 + 0.5, around // 32 + 0.5, 0 * around + 0.5, 0 * around], axis=1).astype(np.float32)
    pts, batch = torch.from_numpy(pts).cuda(), torch.zeros(len(around), dtype=torch.int32, device="cuda")
    assert len(around) > 1024
    a, b = _Bufs(large, 1, 1, 4096), _Bufs(large, 1, 1, 4096)
    _sites(a.ctx, "voxelize", np.sort(np.concatenate([line, around])), large)
    _sites(a.ctx, "voxelize", _small_sites(words, False), (32, words, 1))
    b.call_by_call(pts, batch, spec)
    B.build_stacks((B.StackC * 1)(a.stack(spec, batch)), 1, pts)
    a.ctx.status_sync(), b.ctx.status_sync()
    _same(a, b, f"{large} after {words} words")
    a.ctx.close(), b.ctx.close()


def _index_is(ctx, coords, n, cap, grid):
    """The index in slot 0 against one rebuilt from the coordinates."""
    nbr, ref = (torch.zeros((27, cap), dtype=torch.int32, device="cuda") for _ in range(2))
    ctx.build_kmap(B.SUBM, coords, n, cap, grid, 1, cap, nbr, n, in_slot=0)
    ctx.build_kmap(B.SUBM, coords, n, cap, grid, 1, cap, ref, n)
    ctx.status_sync()
    m = int(n.item())
    assert torch.equal(nbr[:, :m], ref[:, :m])


# Dense grids: bits in the slot instead of marks, a launch more.  Both sides of the lines at 8 192 and 65 536 points, of 2 and 24 cells a point;
# grids of up to 8 192 words (one block) and more.
@pytest.mark.parametrize("n,words,launches", [(8191, 2, 4), (8192, 2, 5), (8192, 512, 5), (8192, 513, 4), (65535, 4095, 5), (65535, 4096, 4),
                                              (65536, 4097, 5), (65536, 8193, 6), (65536, 49152, 6), (65536, 49153, 5), (300001, 2100, 5)])
def test_voxelize_dense_and_sparse_grids(n, words, launches):
    grid = (32, words, 1)
    rng = np.random.RandomState(n + words)
    spec = VoxelSpec((0.0, 0.0, 0.0), (1.0, 1.0, 1.0), grid)
    ctx = B.Context(n, n, 32 * max(words, 60000), n_slots=1)
    _sites(ctx, "voxelize", np.arange(0, 32 * 60000, 300), (32, 60000, 1))        # what the slot holds before
    i32 = dict(dtype=torch.int32, device="cuda")
    for part in (1.0, 0.3):                      # the whole of the grid, then a part: lines that hold nothing any more
        pts = np.stack([rng.uniform(0, 32, n), rng.uniform(0, part * words, n), rng.uniform(0, 1, n), rng.uniform(0, 1, n)], axis=1).astype(np.float32)
        pts[::97, 0] = -1.0                      # dropped
        dev = torch.from_numpy(pts).cuda()
        coords, feats, counts, nv = torch.zeros((n, 4), **i32), torch.ones((n, 4), device="cuda"), torch.ones(n, **i32), torch.zeros(1, **i32)
        call = lambda: ctx.voxelize(dev, None, spec, n, coords, feats, counts, nv)
        call()
        ctx.status_sync()
        oc, om, on = oracle.voxelize(pts, None, spec.lo, spec.vs, spec.grid)
        m = len(oc)
        assert int(nv.item()) == m and np.array_equal(coords[:m].cpu().numpy(), oc) and np.array_equal(counts[:m].cpu().numpy(), on)
        # sums of k points in fp32 against fp64: k * 2^-24 relative to the largest partial sum
        assert_features_close(feats[:m].cpu().numpy(), om, max(4e-6, int(on.max()) * 2.0 ** -24), "means")
        assert not feats[m:].any() and not counts[m:].any()
        _index_is(ctx, coords, nv, n, grid)
    assert _kernels_in(call) == launches
    ctx.close()


# Lines at 180 000 pixels and of pixels^2 / 2^18 cells of the image's frame.
@pytest.mark.parametrize("h,w,grid,nb,launches", [(400, 449, (128, 128, 7), 1, 7), (400, 450, (128, 128, 7), 1, 8), (400, 450, (128, 128, 8), 1, 7),
                                                  (512, 512, (128, 128, 16), 1, 8), (512, 512, (128, 128, 16), 3, 9), (512, 512, (128, 128, 17), 1, 8),
                                                  (700, 1000, (256, 256, 28), 1, 9), (700, 1000, (256, 256, 29), 1, 8)])
def test_pool_dense_and_sparse_grids(h, w, grid, nb, launches):
    rng = np.random.RandomState(h + grid[2])
    npix, bi = h * w, nb - 1
    spec = VoxelSpec((0.0, 0.0, 0.0), (w / grid[0], h / grid[1], 1.0), grid, nb)
    ctx = B.Context(npix, npix, max(cells_of(grid, nb), 32 * 60000), n_slots=1)
    _sites(ctx, "voxelize", np.arange(0, 32 * 60000, 300), (32, 60000, 1))
    q = [1, 0, 0, 0.5, 0, 1, 0, 0.5, 0, 0, 0, 0.5]
    i32 = dict(dtype=torch.int32, device="cuda")
    for rows in (h, h // 4):
        depth = np.zeros((h, w), np.float32)
        depth[:rows] = rng.randint(0, 8, (rows, w)) != 0
        img = rng.randint(-40, 40, (h, w, 8)).astype(np.float16)
        dimg, ddep = torch.from_numpy(img).cuda(), torch.from_numpy(depth).cuda()
        coords, feats, counts, n = torch.zeros((npix, 4), **i32), torch.zeros((npix, 8), dtype=torch.float16, device="cuda"), torch.zeros(npix, **i32), torch.zeros(1, **i32)
        call = lambda: ctx.pool_image(dimg, ddep, q, spec, B.POOL_MAX, npix, coords, feats, counts, n, batch_index=bi)
        call()
        ctx.status_sync()
        oc, of, on = oracle.pool_image(img, depth, q, spec.lo, spec.vs, spec.grid, oracle.POOL_MAX, nb, bi)
        m = len(oc)
        assert int(n.item()) == m and np.array_equal(coords[:m].cpu().numpy(), oc) and np.array_equal(counts[:m].cpu().numpy(), on)
        assert np.array_equal(feats[:m].float().cpu().numpy(), of)
        if nb == 1:
            _index_is(ctx, coords, n, npix, grid)
    assert _kernels_in(call) == launches
    ctx.close()


@pytest.mark.parametrize("n,grid,launches", [(500, (64, 50, 40), 4), (524288, (4096, 4096, 16), 7)])      # marks; counts of the bins
def test_clearing_recorded_after_a_failed_call(n, grid, launches):
    """A call that reports a failed launch may leave scratch behind that is not zero.  Until a launch that clears it has been issued every call
    brings one; one that was recorded into a graph does not count, as nobody may ever replay it."""
    hip = B.load_library()                        # (links the runtime)
    rng = np.random.RandomState(n)
    spec = VoxelSpec((0.0, 0.0, 0.0), (1.0, 1.0, 1.0), grid)
    pts = torch.from_numpy((rng.uniform(0, 1, (n, 4)) * np.array(grid + (1,))).astype(np.float32)).cuda()
    ctx = B.Context(n, n, cells_of(grid, 1), n_slots=1)
    i32 = dict(dtype=torch.int32, device="cuda")
    out, nv = [torch.zeros((n, 4), **i32), torch.zeros((n, 4), device="cuda"), torch.zeros(n, **i32)], torch.zeros(1, **i32)
    call = lambda: ctx.voxelize(pts, None, spec, n, *out, nv)
    call()
    torch.cuda.synchronize()
    want = [t.clone() for t in (*out, nv)]
    assert _kernels_in(call) == launches
    assert hip.hipSetDevice(9999) != 0            # an error of the runtime, left for the next who asks
    with pytest.raises(B.Emc2Error) as e:
        call()
    assert e.value.status == B.ERR_DEVICE
    assert _kernels_in(call) == launches + 1 and _kernels_in(call) == launches + 1
    for t in (*out, nv):
        t.fill_(-3)
    call()
    torch.cuda.synchronize()
    m = int(nv.item())                            # (rows of coordinates beyond the count are not written)
    assert torch.equal(nv, want[3]) and torch.equal(out[0][:m], want[0][:m]) and torch.equal(out[2], want[2])
    assert _kernels_in(call) == launches
    ctx.close()


# runs of sites in one word: whole words, words of every second cell, runs over the ends of rows and of waves; in key order and not
@pytest.mark.parametrize("shuffled", [False, True])
@pytest.mark.parametrize("nl,ni", [(1, 1), (63, 65), (3000, 4097)])
def test_fuse_sites_by_the_word(nl, ni, shuffled):
    grid = (45, 50, 7)
    gx, gy, _ = grid
    rng = np.random.RandomState(nl)
    kl, ki = np.arange(100, 100 + nl), np.arange(7, 7 + 2 * ni, 2)
    if shuffled:
        kl, ki = rng.permutation(kl), rng.permutation(ki)
    ki = ki[ki < int(np.prod(grid))]
    cap = len(kl) + len(ki)
    ctx = B.Context(cap, cap, cells_of(grid, 1), n_slots=1)

    def site(k):
        return torch.from_numpy(np.stack([0 * k, k // (gx * gy), k // gx % gy, k % gx], axis=1).astype(np.int32)).cuda()

    def value(k, c):
        return torch.from_numpy(((k[:, None] * 3 + np.arange(c)) % 997).astype(np.float16)).cuda()

    def count(v):
        return torch.tensor([v], dtype=torch.int32, device="cuda")

    out, n = torch.zeros((cap, 4), dtype=torch.int32, device="cuda"), count(0)
    feats = torch.zeros((cap, 24), dtype=torch.float16, device="cuda")
    for _ in range(2):                   # the second finds the marks as the first left them
        ctx.fuse(F16, site(kl), value(kl, 8), count(len(kl)), len(kl), site(ki), value(ki, 16), count(len(ki)), len(ki), grid, 1, cap, out, feats,
                 n, out_slot=0)
        ctx.status_sync()
        union = np.union1d(kl, ki)
        m = int(n.item())
        assert m == len(union) and np.array_equal(out[:m].cpu().numpy(), site(union).cpu().numpy())
        want = np.zeros((m, 24), np.float16)
        want[np.searchsorted(union, kl), :8], want[np.searchsorted(union, ki), 8:] = value(kl, 8).cpu(), value(ki, 16).cpu()
        assert np.array_equal(feats[:m].cpu().numpy(), want)
    ctx.close()
