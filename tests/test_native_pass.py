"""Argument blocks of a native pass without a GPU: host tensors that call themselves device tensors stand in for the buffers,
and the two native calls record what they are handed, so what a pass passes on, keeps and refuses can be seen."""
import ctypes
import os
import sys

import pytest
import torch

sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))

from paper_2507_04123_amd import binding as B  # noqa: E402
from paper_2507_04123_amd import pipeline as P  # noqa: E402
from paper_2507_04123_amd.configs import F16, Branch, Layer, STRIDED, SUBM, VoxelSpec  # noqa: E402


class _Dev(torch.Tensor):
    is_cuda = True


def _dev(t):
    return None if t is None else t.as_subclass(_Dev)


def _on_device(r):
    """The runner with every buffer on the "device"."""
    for name in ("feats32", "counts", "feats_lp"):
        setattr(r, name, _dev(getattr(r, name)))
    for lv in r.levels:
        for name in ("coords", "n", "subm_nbr", "down_nbr"):
            setattr(lv, name, _dev(getattr(lv, name)))
    r.acts = [_dev(t) for t in r.acts]
    r.wdev = [(_dev(w), lay) for w, lay in r.wdev]
    r.params = [{k: _dev(t) for k, t in p.items()} for p in r.params]
    return r


class _Ctx:
    """What a runner asks of its context."""
    made = 0

    def __init__(self, *a, **k):
        _Ctx.made += 1
        self.h = ctypes.c_void_p(4096 * _Ctx.made)
        self.calls = []

    def uses_mfma(self, dtype, cin, cout):
        return False

    def __getattr__(self, name):
        return lambda *a, **k: self.calls.append((name, a, k))


@pytest.fixture
def native(monkeypatch):
    """The stacks and convolution calls of every pass, copied when they are issued."""
    seen = {"stacks": [], "convs": []}
    monkeypatch.setattr(B, "Context", _Ctx)
    monkeypatch.setattr(B, "build_stacks", lambda st, n, pts: seen["stacks"].append((B.StackC * n).from_buffer_copy(st)))
    monkeypatch.setattr(B, "spconv_list", lambda c, n: seen["convs"].append((B.ConvCallC * n).from_buffer_copy(c)))
    return seen


def _branch(n_levels=2, nb=2):
    layers = [Layer(SUBM, 4, 16)]
    for _ in range(n_levels - 1):
        layers += [Layer(STRIDED, 16, 16), Layer(SUBM, 16, 16)]
    return Branch("b", VoxelSpec((0.0, 0.0, 0.0), (1.0, 1.0, 1.0), (32, 16, 8), nb), tuple(layers))


def _routed(n_levels=2, n=64):
    rr = P.RoutedRunner([_branch(n_levels) for _ in range(3)], F16, n, 2, seed=1, device="cpu")
    for _, r in rr.runners:
        _on_device(r)
    rr.group_batch = [_dev(t) for t in rr.group_batch]
    args = (_dev(torch.zeros((n, 4))), None, torch.zeros((1, 4)), None, 23.5, 0.5)
    return rr, args


def _runner(n=64):
    return _on_device(P.BranchRunner(_Ctx(), _branch(), F16, n, P.device_params(_branch().layers, 1, F16), device="cpu"))


@pytest.fixture(autouse=True)
def _host_params(monkeypatch):
    real = P.device_params
    monkeypatch.setattr(P, "device_params", lambda layers, seed, dtype: real(layers, seed, dtype, device="cpu"))


def test_routed_pass_hands_on_the_routing_it_holds(native):
    """The stacks are routed by the tensors that this pass's dispatcher and grouping write, not by an earlier pass's."""
    rr, args = _routed()
    rr.run(*args)
    kept = rr.expert, rr.slot                    # an earlier pass's routing, kept by the caller
    for name in ("expert", "slot"):
        setattr(rr, name, torch.zeros_like(getattr(rr, name)))
        rr.run(*args)
        for s in native["stacks"][-1]:
            assert (s.d_route, s.d_slot) == (rr.expert.data_ptr(), rr.slot.data_ptr())
    assert native["stacks"][0][0].d_route == kept[0].data_ptr() != rr.expert.data_ptr()


def _same(a, b):
    return bytes(a) == bytes(b)


def test_kept_blocks_follow_everything_that_went_into_them(native):
    """A level's capacity is the pitch of its maps for the stacks and for the convolutions; rows, layouts and types count as
    addresses do; what has not changed is not filled again."""
    r, pts = _runner(), _dev(torch.zeros((64, 4)))

    def both():
        r.run(pts, None)
        return native["stacks"][-1][0], native["convs"][-1]

    s0, c0 = both()
    blocks = r.native.calls
    s1, c1 = both()
    assert _same(s0, s1) and _same(c0, c1) and r.native.calls is blocks
    r.levels[1].cap -= 5
    s1, c1 = both()
    assert s1.level[1].capacity == s0.level[1].capacity - 5
    assert [c.capacity_out for c in c1] == [c0[0].capacity_out, c0[1].capacity_out - 5, c0[2].capacity_out - 5]
    r.levels[1].cap += 5
    full, r.acts[0] = r.acts[0], r.acts[0][:40]            # the same address, fewer rows that a map entry may name
    with pytest.raises(ValueError, match="smaller than capacity"):
        r.run(pts, None)                                   # it is also an output of 64 rows
    r.acts[0] = full
    r.feats_lp, full = r.feats_lp[:40], r.feats_lp
    assert r.native.convs((r,)) and native["convs"][-1][0].n_in_rows == 40
    r.feats_lp = full
    r.wdev[2] = (r.wdev[2][0], B.W_PACKED)
    assert [c.w_layout for c in both()[1]] == [B.W_PLAIN, B.W_PLAIN, B.W_PACKED]
    r.acts[1] = r.acts[1].view(torch.bfloat16)             # the same address, another type
    for _ in range(2):
        with pytest.raises(ValueError, match="out"):
            r.run(pts, None)


def _host(t):
    return t.as_subclass(torch.Tensor)


# a buffer in turn: half its rows, another type of the same width, every second row of a larger one, on the host
@pytest.mark.parametrize("name", ["feats32", "counts", "feats_lp", "coords", "n", "subm_nbr", "down_nbr"])
def test_maps_refuse_buffers_they_would_write_out_of(native, name):
    r, pts = _runner(), _dev(torch.zeros((64, 4)))
    at = r if hasattr(r, name) else r.levels[1]
    r.run_maps(pts, None)
    good = getattr(at, name)
    bad = [_host(good)]
    if name != "n":
        bad.append(good[: good.shape[0] // 2])
    if name != "feats_lp":                                  # (its type may be either of two, and it may lie apart)
        bad += [good.view(torch.float32 if good.dtype == torch.int32 else torch.int32), torch.cat([good, good])[::2]]
        if name == "n":
            bad.pop()                                       # one element is contiguous whatever its stride
    issued = len(native["stacks"])
    for t in bad:
        setattr(at, name, t)
        for _ in range(2):                                  # refused each time, not only by the pass that meets it first
            with pytest.raises(ValueError):
                r.run_maps(pts, None)
        with pytest.raises(ValueError):
            r.run(pts, None)
    assert len(native["stacks"]) == issued
    setattr(at, name, good)
    r.run_maps(pts, None)


def test_maps_refuse_frame_ids_and_grids_that_do_not_fit(native):
    r, pts, ids = _runner(), _dev(torch.zeros((64, 4))), _dev(torch.zeros(64, dtype=torch.int32))
    r.run_maps(pts, ids)
    assert native["stacks"][-1][0].d_batch == ids.data_ptr()
    for p, b in ((pts, ids[:63]), (pts, ids.long()), (pts, _host(ids)), (pts.view(-1), _dev(torch.zeros(256, dtype=torch.int32)))):
        with pytest.raises(ValueError):
            r.run_maps(p, b)
    r.levels[1].grid = (1, 2, 3)
    with pytest.raises(B.Emc2Error):
        r.run_maps(pts, ids)
    assert len(native["stacks"]) == 1


def test_routed_pass_of_stacks_with_six_levels_goes_call_by_call(native):
    """Stacks that one native call does not cover: grouped and run one expert after the other."""
    rr, args = _routed(n_levels=6)
    outs = rr.run(*args)
    assert not native["stacks"] and len(outs) == 3
    names = [[c[0] for c in ctx.calls] for ctx, _ in rr.runners]
    assert names[0][:2] == ["dispatch", "group_points"]
    for e, (ctx, r) in enumerate(rr.runners):
        i = names[e].index("group_points")
        assert ctx.calls[i][1][6] == e and ctx.calls[i][1][8] is rr.group_batch[e]
        assert names[e][i + 1] == "voxelize" and ctx.calls[i + 1][1][1] is rr.group_batch[e]
        assert names[e].count("build_kmap") == 11 and names[e].count("spconv") == 11


def test_routed_pass_writes_the_batch_ids_it_used(native):
    rr, args = _routed()
    rr.run(*args)
    assert [s.d_group_batch for s in native["stacks"][-1]] == [t.data_ptr() for t in rr.group_batch]
    rr.group_batch[1] = _dev(torch.zeros(64, dtype=torch.int32))
    rr.run(*args)
    assert native["stacks"][-1][1].d_group_batch == rr.group_batch[1].data_ptr()
    rr.group_batch[1] = _dev(torch.zeros(63, dtype=torch.int32))
    with pytest.raises(ValueError, match="group_batch"):
        rr.run(*args)
