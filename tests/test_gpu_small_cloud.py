"""A small cloud on a small grid: the whole stack in one launch against the calls it replaces, at the edges of its range; and the fp32
convolution with four threads a row against the one with a thread a row."""
import numpy as np
import pytest
import torch

from paper_2507_04123_amd import binding as B
from paper_2507_04123_amd.configs import EPI_AFFINE, EPI_AFFINE_RELU, EPI_NONE, F32, VoxelSpec
from test_gpu_stacks import _Bufs, _kernels_in, _points, _same

pytestmark = pytest.mark.gpu


def _crowd(pts, batch, grid, seed):
    """Voxels of 2, 4, 5 and 300 points in the last frame, the grid's first and last cells among them; the others hold one."""
    rng = np.random.RandomState(seed)
    nb = int(batch.max().item()) + 1
    at = 0
    for k, cell in ((2, (0, 0, 0)), (4, (grid[0] - 1, grid[1] - 1, grid[2] - 1)), (5, (1, 0, 0)), (300, (grid[0] - 1, 0, grid[2] - 1))):
        xyz = np.array(cell) + rng.uniform(0.1, 0.9, (k, 3))
        pts[at:at + k, :3] = torch.from_numpy(xyz.astype(np.float32)).cuda()
        batch[at:at + k] = nb - 1
        at += k


@pytest.mark.parametrize("n", [1024, 1025, 2047, 9000, 15360, 15361])
@pytest.mark.parametrize("grid,nb", [((50, 131, 40), 1), ((31, 33, 17), 3), ((64, 64, 16), 4)])
def test_one_launch_equals_the_calls(n, grid, nb):
    spec = VoxelSpec((0.0, 0.0, 0.0), (1.0, 1.0, 1.0), grid, nb)
    a, b = _Bufs(grid, nb, 1, n), _Bufs(grid, nb, 1, n)
    for k in range(3):                            # later passes meet an index that holds the bits of the one before
        pts, batch = _points(n + k, grid, nb, n)
        if k:
            _crowd(pts, batch, grid, k)
        a.feats.fill_(5.0), a.counts.fill_(5), b.feats.fill_(5.0), b.counts.fill_(5)
        b.call_by_call(pts, batch, spec)
        arr = (B.StackC * 1)(a.stack(spec, batch))
        B.build_stacks(arr, 1, pts)
        torch.cuda.synchronize()
        a.ctx.status_sync(); b.ctx.status_sync()
        m = int(b.n[0].item())
        if k:                                     # more than four points are summed in an order of their own: 300 * 2^-24
            many = b.counts > 4
            assert torch.allclose(a.feats, b.feats, rtol=2e-5)
            a.feats[many], a.lp[many] = b.feats[many], b.lp[many]
        _same(a, b, f"{n} points, pass {k}")
        assert not a.feats[m:].any() and not a.counts[m:].any()
    assert _kernels_in(lambda: B.build_stacks(arr, 1, pts)) == (1 if n <= 15360 else 5)
    again = torch.full_like(a.subm[0], -9)        # the slot holds the index
    a.ctx.build_kmap(B.SUBM, a.coords[0], a.n[0], a.cap[0], grid, nb, a.cap[0], again, a.n[0], in_slot=0)
    assert torch.equal(again[:, :m], b.subm[0][:, :m])
    a.ctx.close(); b.ctx.close()


def test_one_launch_of_several_stacks_and_capacity():
    n = 3000
    grids = [(50, 131, 40), (25, 66, 20), (13, 33, 10)]
    pts, batch = _points(1, grids[0], 1, n)
    specs = [VoxelSpec((0.0, 0.0, 0.0), (s, s, s), g) for s, g in zip((1.0, 2.0, 4.0), grids)]
    a, b = [_Bufs(g, 1, 1, n) for g in grids], [_Bufs(g, 1, 1, n) for g in grids]
    arr = (B.StackC * 3)(*[x.stack(s, batch) for x, s in zip(a, specs)])
    B.build_stacks(arr, 3, pts)
    for x, y, s in zip(a, b, specs):
        y.call_by_call(pts, batch, s)
        torch.cuda.synchronize()
        few = y.counts <= 4
        assert torch.allclose(x.feats, y.feats, rtol=1e-5)
        x.feats[~few], x.lp[~few] = y.feats[~few], y.lp[~few]
        _same(x, y, str(s))
    arr[0].level[0].capacity = 1000               # fewer than there are voxels
    a[0].coords[0][1000:] = -5
    B.build_stacks(arr, 1, pts)
    with pytest.raises(B.Emc2Error) as e:
        a[0].ctx.status_sync()
    assert e.value.status == B.ERR_CAPACITY
    assert int(a[0].n[0].item()) == 1000 and torch.equal(a[0].coords[0][:1000], b[0].coords[0][:1000])
    assert torch.equal(a[0].feats[:1000], b[0].feats[:1000]) and bool((a[0].coords[0][1000:] == -5).all())
    for x in a + b:
        x.ctx.close()


@pytest.mark.parametrize("cin,cout", [(4, 16), (4, 32), (16, 16)])
@pytest.mark.parametrize("n,epi", [(1, EPI_NONE), (63, EPI_AFFINE), (64, EPI_AFFINE_RELU), (65, EPI_NONE), (5000, EPI_AFFINE_RELU), (65536, EPI_AFFINE)])
def test_four_threads_a_row(cin, cout, n, epi):
    """Both forms add in one order: the same bits."""
    g = torch.Generator(device="cuda").manual_seed(n + cin)
    x = torch.randn((n, cin), generator=g, device="cuda")
    w = torch.randn((27, cin, cout), generator=g, device="cuda") * 0.1
    sc, sh = (torch.rand(cout, generator=g, device="cuda"), torch.randn(cout, generator=g, device="cuda")) if epi != EPI_NONE else (None, None)
    ctx = B.Context(16, 16, 64, n_slots=1)
    nn = torch.tensor([n], dtype=torch.int32, device="cuda")
    ys = []
    for cap in (n, 65537):
        nbr = torch.randint(-n, n, (27, cap), generator=torch.Generator(device="cuda").manual_seed(3), device="cuda", dtype=torch.int32)
        if ys:
            nbr[:, :n] = first
        else:
            first = nbr[:, :n].clone()
        y = torch.full((cap, cout), 7.0, device="cuda")
        ctx.spconv(F32, x, w, sc, sh, epi, nbr, nn, cap, y)
        ctx.status_sync()
        assert bool((y[n:] == 7.0).all())
        ys.append(y[:n])
    assert torch.equal(ys[0], ys[1])
    ref = torch.zeros((n, cout), dtype=torch.float64, device="cuda")
    for k in range(27):
        have = first[k] >= 0
        ref[have] += x[first[k][have].long()].double() @ w[k].double()
    if epi != EPI_NONE:
        ref = ref * sc.double() + sh.double()
    if epi == EPI_AFFINE_RELU:
        ref = ref.clamp(min=0)
    # fp32 sums of at most 27 * 16 products: well inside 27 * 16 * 2^-24 of the sum of magnitudes
    assert float((ys[0].double() - ref).abs().max()) <= 3e-5 * float(ref.abs().max() + 1)
    ctx.close()
