"""GPU tests of emc2_build_stacks (all levels of several stacks in one call) against emc2_voxelize + emc2_build_kmap, which
are held to the oracle elsewhere: coordinates, counts, means, kernel maps and index slots, bit for bit (voxels of at most
four points, so the means are exact too)."""
import numpy as np
import pytest
import torch

from paper_2507_04123_amd import binding as B
from paper_2507_04123_amd.configs import VoxelSpec, out_grid
from paper_2507_04123_amd.pipeline import cells_of

pytestmark = pytest.mark.gpu


def _points(seed, grid, nb, n):
    """At most one point per cell and frame on average half of the cells' rows, a few outside the grid and with bad frame ids."""
    rng = np.random.RandomState(seed)
    cells = grid[0] * grid[1] * grid[2]
    pick = rng.choice(cells * nb, min(n, cells * nb), replace=False)
    b, k = pick // cells, pick % cells
    xyz = np.stack([k % grid[0], k // grid[0] % grid[1], k // (grid[0] * grid[1])], 1) + rng.uniform(0.1, 0.9, (len(pick), 3))
    pts = np.concatenate([xyz, rng.uniform(0, 1, (len(pick), 1))], 1).astype(np.float32)
    pts[::17, 0] -= 2 * grid[0]                   # outside
    b = b.astype(np.int32)
    b[::23] = -1                                  # dropped
    return torch.from_numpy(pts).cuda(), torch.from_numpy(b).cuda()


class _Bufs:
    def __init__(self, grid, nb, n_levels, n_points):
        self.grids, self.cap = [grid], []
        for _ in range(n_levels - 1):
            self.grids.append(out_grid(self.grids[-1]))
        i32 = dict(dtype=torch.int32, device="cuda")
        prev = n_points
        self.coords, self.n, self.subm, self.down = [], [], [], []
        for l, g in enumerate(self.grids):
            cap = min(prev if l == 0 else 8 * prev, cells_of(g, nb))
            prev = cap
            self.cap.append(cap)
            self.coords.append(torch.full((cap, 4), -9, **i32))
            self.n.append(torch.full((1,), -9, **i32))
            self.subm.append(torch.full((27, cap), -9, **i32))
            self.down.append(torch.full((27, cap), -9, **i32) if l else None)
        c0 = self.cap[0]
        self.feats, self.counts = torch.zeros((c0, 4), device="cuda"), torch.zeros((c0,), **i32)
        self.lp = torch.zeros((c0, 4), dtype=torch.float16, device="cuda")
        self.ctx = B.Context(max(n_points, 1), max(self.cap), cells_of(grid, nb), n_slots=n_levels)

    def stack(self, spec, batch):
        s = B.StackC()
        s.ctx, s.spec, s.expert, s.n_levels, s.lp_dtype = self.ctx.h, B.voxel_spec_c(spec, 4), -1, len(self.grids), B.F16
        s.d_batch = batch.data_ptr()
        s.d_feats, s.d_counts, s.d_feats_lp = self.feats.data_ptr(), self.counts.data_ptr(), self.lp.data_ptr()
        for l in range(len(self.grids)):
            c = s.level[l]
            c.capacity, c.slot, c.d_coords, c.d_n = self.cap[l], l, self.coords[l].data_ptr(), self.n[l].data_ptr()
            c.d_subm_nbr, c.d_down_nbr = self.subm[l].data_ptr(), (self.down[l].data_ptr() if l else None)
        return s

    def call_by_call(self, pts, batch, spec):
        ctx, nb = self.ctx, spec.n_batch
        ctx.voxelize(pts, batch, spec, self.cap[0], self.coords[0], self.feats, self.counts, self.n[0], feats_lp=self.lp, index_slot=0)
        for l in range(len(self.grids)):
            if l:
                ctx.build_kmap(B.STRIDED, self.coords[l - 1], self.n[l - 1], self.cap[l - 1], self.grids[l - 1], nb, self.cap[l],
                               self.down[l], self.n[l], out_coords=self.coords[l], in_slot=l - 1, out_slot=l)
            ctx.build_kmap(B.SUBM, self.coords[l], self.n[l], self.cap[l], self.grids[l], nb, self.cap[l], self.subm[l], self.n[l], in_slot=l)


def _same(a, b, what):
    for l in range(len(a.grids)):
        n = int(b.n[l].item())
        assert int(a.n[l].item()) == n, f"{what} level {l}: count"
        assert torch.equal(a.coords[l][:n], b.coords[l][:n]), f"{what} level {l}: coordinates"
        assert torch.equal(a.subm[l][:, :n], b.subm[l][:, :n]), f"{what} level {l}: submanifold map"
        if l:
            assert torch.equal(a.down[l][:, :n], b.down[l][:, :n]), f"{what} level {l}: stride-2 map"
    n0 = int(b.n[0].item())
    for t, u, nm in ((a.feats, b.feats, "means"), (a.counts, b.counts, "counts"), (a.lp, b.lp, "fp16 means")):
        assert torch.equal(t[:n0], u[:n0]), f"{what}: {nm}"


# grids whose rows are shorter than a word, straddle words, fill lines exactly, and leave a lone output column; one level to
# five; batches; more than one granule (4 096 coarse cells) and tile (65 536 cells); a level 1 of large granules (4.5 million
# cells) over a level 2 of small ones
@pytest.mark.parametrize("grid,nb,levels,n", [((7, 5, 3), 1, 3, 40), ((3, 9, 6), 3, 2, 200), ((1, 1, 1), 2, 1, 2), ((33, 17, 9), 2, 4, 900),
                                              ((64, 16, 4), 1, 2, 500), ((65, 40, 11), 2, 5, 3000), ((176, 200, 5), 1, 4, 6000),
                                              ((513, 300, 3), 2, 3, 20000), ((1, 700, 90), 1, 3, 5000),
                                              ((1408, 800, 32), 1, 3, 20000)])
def test_stack_equals_the_calls_it_replaces(grid, nb, levels, n):
    spec = VoxelSpec((0.0, 0.0, 0.0), (1.0, 1.0, 1.0), grid, nb)
    a, b = _Bufs(grid, nb, levels, n), _Bufs(grid, nb, levels, n)
    for k in range(3):                            # later passes meet an index that holds the bits of the one before
        pts, batch = _points(10 * n + k, grid, nb, n if k != 1 else max(1, n // 9))
        b.call_by_call(pts, batch, spec)
        B.build_stacks((B.StackC * 1)(a.stack(spec, batch)), 1, pts)
        torch.cuda.synchronize()
        a.ctx.status_sync(); b.ctx.status_sync()
        _same(a, b, f"{grid} x{nb} pass {k}")
    # the slots hold the levels' indexes: a map built from them alone
    l = levels - 1
    again = torch.full_like(a.subm[l], -9)
    a.ctx.build_kmap(B.SUBM, a.coords[l], a.n[l], a.cap[l], a.grids[l], nb, a.cap[l], again, a.n[l], in_slot=l)
    m = int(a.n[l].item())
    assert torch.equal(again[:, :m], b.subm[l][:, :m])
    a.ctx.close(); b.ctx.close()


def test_several_stacks_in_one_call_and_their_errors():
    specs = [(VoxelSpec((0.0, 0.0, 0.0), (1.0, 1.0, 1.0), (60, 50, 10), 2), 3), (VoxelSpec((0.0, 0.0, 0.0), (2.0, 2.0, 2.0), (30, 25, 5), 2), 1),
             (VoxelSpec((0.0, 0.0, 0.0), (4.0, 4.0, 4.0), (15, 13, 3), 2, 0.0, 900.0), 4)]
    pts, batch = _points(3, (60, 50, 10), 2, 4000)
    many = [_Bufs(s.grid, 2, lv, 4000) for s, lv in specs]
    ref = [_Bufs(s.grid, 2, lv, 4000) for s, lv in specs]
    arr = (B.StackC * 3)(*[m.stack(s, batch) for m, (s, _) in zip(many, specs)])
    for k in range(2):
        B.build_stacks(arr, 3, pts)
    for m, r, (s, _) in zip(many, ref, specs):
        r.call_by_call(pts, batch, s)
        torch.cuda.synchronize()
        for l in range(len(m.grids)):
            nl = int(r.n[l].item())
            assert int(m.n[l].item()) == nl and torch.equal(m.coords[l][:nl], r.coords[l][:nl])
            assert torch.equal(m.subm[l][:, :nl], r.subm[l][:, :nl])
    arr[1].ctx = arr[0].ctx
    with pytest.raises(B.Emc2Error, match="one context"):
        B.build_stacks(arr, 3, pts)
    arr[1].ctx = many[1].ctx.h
    arr[0].level[1].slot = 0
    with pytest.raises(B.Emc2Error, match="share slot"):
        B.build_stacks(arr, 3, pts)
    arr[0].level[1].slot, arr[0].level[1].capacity = 1, 5       # more outputs than capacity: reported, in bounds
    B.build_stacks(arr, 1, pts)
    torch.cuda.synchronize()
    assert int(many[0].n[1].item()) == 5
    with pytest.raises(B.Emc2Error) as ei:
        many[0].ctx.status_sync()
    assert ei.value.status == B.ERR_CAPACITY
    for m in many + ref:
        m.ctx.close()


def test_a_refused_call_leaves_every_slot_as_it_was():
    spec, (pts, batch) = VoxelSpec((0.0, 0.0, 0.0), (1.0, 1.0, 1.0), (20, 10, 4), 2), _points(5, (20, 10, 4), 2, 300)
    bufs = [_Bufs(spec.grid, 2, 2, 300) for _ in range(2)]
    arr = (B.StackC * 2)(*[b.stack(spec, batch) for b in bufs])
    arr[1].level[1].slot = 7                      # the second stack's fault: the first one is not built either
    with pytest.raises(B.Emc2Error, match="slot"):
        B.build_stacks(arr, 2, pts)
    a = bufs[0]
    a.n[0].zero_()
    with pytest.raises(B.Emc2Error):              # no index there to build a map from
        a.ctx.build_kmap(B.SUBM, a.coords[0], a.n[0], a.cap[0], spec.grid, 2, a.cap[0], a.subm[0], a.n[0], in_slot=0)
    for b in bufs:
        b.ctx.close()


class _Timer:
    """A timer makes a runner issue its pass call by call."""

    def __call__(self, tag):
        return self

    def __enter__(self):
        return self

    def __exit__(self, *exc):
        return False


def _runner(n):
    import dataclasses
    from paper_2507_04123_amd.configs import get_config
    from paper_2507_04123_amd.pipeline import ConfigRunner
    cfg = get_config(2)
    return ConfigRunner(dataclasses.replace(cfg, n_points=n, n_frames=1), n)


def test_pass_follows_what_its_runner_holds():
    """A pass works on the tensors and the context that the runner holds when it is issued, checks what it has not seen
    before, takes a frame without points, and refuses a closed context."""
    from paper_2507_04123_amd import gen
    from paper_2507_04123_amd.configs import get_config
    n = 4000
    cr = _runner(n)
    ctx, r = cr.branches[0]
    pts = torch.from_numpy(gen.make_frames(get_config(2))[0][::30][:n]).cuda().contiguous()
    first = cr.run(pts, None)[0].clone()
    k = len(r.params) - 1
    r.params[k]["scale"] = r.params[k]["scale"] * 2.0       # the tensor that the first pass read is gone
    r.acts[k - 1] = torch.zeros_like(r.acts[k - 1])
    torch.cuda.empty_cache()
    got = cr.run(pts, None)[0].clone()
    single = r.run(pts, None).clone()
    m = int(r.levels[-1].n.item())
    want = cr.run(pts, None, timer=_Timer())[0]
    assert torch.equal(got[:m], want[:m]) and torch.equal(single[:m], want[:m]) and not torch.equal(got[:m], first[:m])
    good, r.params[k]["scale"] = r.params[k]["scale"], r.params[k]["scale"].cpu()
    for _ in range(2):                                      # refused each time, not only by the pass that meets it first
        with pytest.raises(ValueError, match="scale"):
            cr.run(pts, None)
    r.params[k]["scale"] = good
    cr.run(pts[:0], None)
    ctx.status_sync()
    assert all(int(lv.n.item()) == 0 for lv in r.levels)
    assert torch.equal(cr.run(pts, None)[0][:m], got[:m])
    ctx.status_sync()
    ctx.close()
    with pytest.raises(B.Emc2Error):
        cr.run(pts, None)
    with pytest.raises(B.Emc2Error):
        r.run(pts, None)


def test_routed_pass_takes_as_many_points_as_it_was_made_for():
    from paper_2507_04123_amd.configs import F16, expert_branches
    from paper_2507_04123_amd.pipeline import RoutedRunner
    rr = RoutedRunner(expert_branches(2), F16, 512, 2, seed=3)
    pts, scene = torch.zeros((512, 4), device="cuda"), torch.zeros(512, dtype=torch.int32, device="cuda")
    props, prop_scene = torch.ones((1, 4), device="cuda"), torch.zeros(1, dtype=torch.int32, device="cuda")
    rr.run(pts, scene, props, prop_scene, 23.5, 0.5)
    for p, s in ((pts[:500], scene[:500]), (pts, scene[:500]), (pts[:500], None)):
        with pytest.raises(ValueError, match="n_points"):
            rr.run(p, s, props, prop_scene, 23.5, 0.5)
    rr.status_sync()
    rr.close()


@pytest.mark.parametrize("with_scene", [True, False])
def test_routed_pass_writes_the_batch_ids_that_group_points_writes(with_scene):
    """Every point's id, those outside the grid and of malformed scenes included; and stacks of more levels than one call
    takes give the levels they share with shorter ones the same voxels."""
    import dataclasses
    from paper_2507_04123_amd.configs import F16, Layer, STRIDED, SUBM, expert_branches
    from paper_2507_04123_amd.pipeline import RoutedRunner
    n, ns = 3001, 4
    base = [dataclasses.replace(b, layers=b.layers[:1] + (Layer(STRIDED, b.layers[0].cout, 32), Layer(SUBM, 32, 32))) for b in expert_branches(ns)]
    longer = [dataclasses.replace(b, layers=b.layers + (Layer(STRIDED, 32, 32),) * 4) for b in base]
    g = torch.Generator(device="cuda").manual_seed(7)
    pts = torch.rand((n, 4), generator=g, device="cuda") * torch.tensor([80.0, 90.0, 5.0, 1.0], device="cuda") - torch.tensor([5.0, 45.0, 3.5, 0.0], device="cuda")
    scene = torch.randint(-1, ns + 1, (n,), generator=g, device="cuda", dtype=torch.int32) if with_scene else None
    props = torch.tensor([[10.0, 0.0, 0.0, 0.9], [60.0, 0.0, 0.0, 0.9], [10.0, 1.0, 0.0, 0.1], [50.0, 9.0, 0.0, 0.2]], device="cuda")
    pscene = torch.tensor([0, 1, 2, 3], dtype=torch.int32, device="cuda")
    a, b = RoutedRunner(base, F16, n, ns, seed=3), RoutedRunner(longer, F16, n, ns, seed=3)
    assert a.native is not None and b.native is None
    for rr in (a, b):
        rr.run(pts, scene, props, pscene, 23.5, 0.5)
        rr.status_sync()
    ctx = a.runners[0][0]
    seen = set(a.expert.tolist())
    assert len(seen) > 1
    for e, ((_, ra), (_, rb)) in enumerate(zip(a.runners, b.runners)):
        want = torch.full((n,), -7, dtype=torch.int32, device="cuda")
        ctx.group_points(scene, n, a.expert, a.order, a.counts, ns, e, a.slot, want)
        assert torch.equal(a.group_batch[e], want) and torch.equal(b.group_batch[e], want)
        for la, lb in zip(ra.levels, rb.levels):
            m = int(la.n.item())
            assert int(lb.n.item()) == m and torch.equal(la.coords[:m], lb.coords[:m])
    a.close()
    b.close()


def test_a_refused_list_says_why_whatever_went_wrong_before():
    """The text is the failing call's, not an older one of another context in the list."""
    ctx = [B.Context(16, 16, 64, n_slots=1) for _ in range(2)]
    i32 = dict(dtype=torch.int32, device="cuda")
    x, w, y = torch.zeros((16, 4), device="cuda"), torch.zeros((27, 4, 16), device="cuda"), torch.zeros((16, 16), device="cuda")
    nbr, n = torch.full((27, 16), -1, **i32), torch.zeros(1, **i32)
    with pytest.raises(B.Emc2Error, match="n_points"):           # an old error of the first context
        ctx[0].voxelize(torch.zeros((17, 4), device="cuda"), None, VoxelSpec((0.0,) * 3, (1.0,) * 3, (4, 4, 4)), 16,
                        nbr[:4].view(16, 4), x, nbr[0], n)
    calls = (B.ConvCallC * 2)()
    for c, t in zip(calls, ctx):
        c.ctx, c.d_in, c.d_w, c.d_nbr, c.d_n_out, c.d_out = t.h, x.data_ptr(), w.data_ptr(), nbr.data_ptr(), n.data_ptr(), y.data_ptr()
        c.capacity_out, c.n_in_rows, c.dtype, c.map_hint, c.cin, c.cout = 16, 16, B.F32, B.MAP_ANY, 4, 16
    B.spconv_list(calls, 2)
    calls[1].capacity_out = 0
    with pytest.raises(B.Emc2Error, match="capacity_out < 1"):
        B.spconv_list(calls, 2)
    calls[1].ctx = None
    with pytest.raises(B.Emc2Error, match="call 1 has no context"):
        B.spconv_list(calls, 2)
    calls[0].ctx = None
    with pytest.raises(B.Emc2Error, match="closed"):
        B.spconv_list(calls, 2)
    stacks = (B.StackC * 2)()
    stacks[0].ctx = ctx[0].h
    with pytest.raises(B.Emc2Error, match="stack 1 has no context"):
        B.build_stacks(stacks, 2, x)
    for t in ctx:
        t.close()


def _kernels_in(issue):
    """Launches of what `issue` issues: the nodes of a graph that captures it."""
    import ctypes
    graph = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(graph, stream=torch.cuda.Stream()):
        issue()
    count = ctypes.c_size_t(0)
    hip = B.load_library()                        # (links the runtime)
    hip.hipGraphGetNodes.argtypes = [ctypes.c_void_p, ctypes.c_void_p, ctypes.POINTER(ctypes.c_size_t)]
    assert hip.hipGraphGetNodes(graph.raw_cuda_graph(), None, ctypes.byref(count)) == 0
    return count.value


# words of the finest index: one tile of 2 048, a word more, the four tiles that one block takes, a word more
@pytest.mark.parametrize("words,levels,launches", [(2048, 1, 5), (2049, 1, 5), (6250, 1, 5), (8192, 1, 5), (8193, 1, 6), (8192, 2, 6)])
def test_small_index_scanned_by_one_block(words, levels, launches):
    grid = (32, words, 1)
    spec = VoxelSpec((0.0, 0.0, 0.0), (1.0, 1.0, 1.0), grid)
    for n in (3, 700, 8 * words):
        a, b = _Bufs(grid, 1, levels, n), _Bufs(grid, 1, levels, n)
        for k in range(2):
            pts, batch = _points(n + k, grid, 1, n)
            if k:
                pts[:, 1] = words - 0.5           # the last tile alone holds a bit
            b.call_by_call(pts, batch, spec)
            arr = (B.StackC * 1)(a.stack(spec, batch))
            B.build_stacks(arr, 1, pts)
            torch.cuda.synchronize()
            a.ctx.status_sync(); b.ctx.status_sync()
            if k:                                 # (many points to a cell: their means depend on the order)
                m = int(b.n[0].item())
                assert int(a.n[0].item()) == m > 0 and torch.equal(a.coords[0][:m], b.coords[0][:m])
            else:
                _same(a, b, f"{words} words, {n} points")
        assert _kernels_in(lambda: B.build_stacks(arr, 1, pts)) == launches
        a.ctx.close(); b.ctx.close()
