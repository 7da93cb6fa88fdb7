"""GPU tests at the sizes where a launch changes shape: tiles and passes of the span convolution, the grid limit and the two
walks of the register-direct one, rows a wave of the quantised one, vector tails of the quantisers, waves and shared cells of the voxelizer, the three-launch index scan, more pieces of
rows than one step of a copy's threads."""
import os
import re

import numpy as np
import pytest
import torch

import oracle
from paper_2507_04123_amd import binding as B
from paper_2507_04123_amd.configs import BF16, EPI_AFFINE, EPI_AFFINE_RELU, EPI_NONE, F16, VoxelSpec
from paper_2507_04123_amd.pipeline import cells_of

pytestmark = pytest.mark.gpu


def _map(n, seed, shuffled):
    """27 taps over n rows: row o reads rows near o (ascending along the row where valid, as kernel maps are), a third of the
    entries absent; `shuffled` permutes a tap, which no interval of rows covers."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    o = torch.arange(n, device="cuda")
    nbr = torch.stack([o + (k % 3 - 1) + 37 * (k // 3 - 4) for k in range(27)])
    drop = torch.rand((27, n), generator=g, device="cuda") < 1 / 3
    nbr = torch.where((nbr < 0) | (nbr >= n) | drop, torch.full_like(nbr, -1), nbr)
    if shuffled:
        nbr[4] = nbr[4][torch.randperm(n, generator=g, device="cuda")]
    return nbr.to(torch.int32).contiguous()


def _check_conv(n, cin, cout, hint, shuffled, seed=11, cap=None, rows_in=None):
    """n rows of `cap` (the pitch of the map; what lies beyond n is not read for a result), `rows_in` rows vouched for."""
    cap = n if cap is None else cap
    g = torch.Generator(device="cuda").manual_seed(seed)
    x = torch.randn((n, cin), generator=g, device="cuda").half()
    w = (torch.randn((27, cin, cout), generator=g, device="cuda") * 0.1).half()
    nbr = torch.zeros((27, cap), dtype=torch.int32, device="cuda")
    nbr[:, :n] = _map(n, seed, shuffled)
    ctx = B.Context(16, 16, 64, n_slots=1)
    wp = torch.empty_like(w)
    ctx.pack_weights(F16, w, wp)
    y = torch.full((cap + 3, cout), 77.0, dtype=torch.float16, device="cuda")
    ctx.spconv(F16, x, wp, None, None, EPI_NONE, nbr, torch.tensor([n], dtype=torch.int32, device="cuda"), cap, y[:cap],
               w_layout=B.W_PACKED, map_hint=hint, n_in_rows=rows_in)
    ctx.status_sync()
    exp = torch.zeros((n, cout), device="cuda")
    for k in range(27):
        rows = (nbr[k][:n] >= 0).nonzero().squeeze(1)
        exp[rows] += x[nbr[k][rows].long()].float() @ w[k].float()
    # the result is rounded once to fp16 (2^-11 relative); sums of up to 27 * cin fp32 products in another order stay below that
    rms = float(exp.square().mean().sqrt())
    err = (y[:n].float() - exp).abs() - 2.0 ** -10 * (exp.abs() + rms)
    assert float(err.max()) <= 0.0
    assert bool((y[n:] == 77.0).all())
    ctx.close()


# tiles of 192, 256, 320 or 384 rows, 256 of them at a time
@pytest.mark.parametrize("n", [1, 17, 129, 32768, 32769, 65537, 98305, 131071, 131072, 131073, 131072 + 40001, 262144 + 70001,
                               98304, 131072 + 98304, 131072 + 98305, 131072 + 102401, 262144 - 1])
def test_span_conv_rounds(n):
    _check_conv(n, 64, 64, B.SUBM, False)


# a row less than, as many as and a row more than the tiles of a round and the sizes where the tile's height changes
@pytest.mark.parametrize("n", [191, 193, 256 * 192, 256 * 192 + 1, 256 * 256, 256 * 256 + 1, 256 * 320 + 1, 3 * 256 * 384 - 1, 3 * 256 * 320 + 65])
def test_span_conv_tiles(n):
    _check_conv(n, 64, 64, B.SUBM, False)


@pytest.mark.parametrize("n", [1, 63, 65, 256 * 64 + 1, 256 * 128 + 1, 256 * 192, 256 * 192 + 1, 2 * 256 * 192 + 70])
def test_span_conv_tiles_of_128_channels(n):
    _check_conv(n, 128, 128, B.SUBM, n == 65)


# Groups whose rows fit the row buffer, fit it in two halves of a tile, and do not; the bf16 form; a row whose 27 entries
# are all absent; no rows at all; 128 channels, in two passes.  Sums of up to 27 * 128 products, rounded once: 2^-11 (fp16) or 2^-8 (bf16) relative, doubled.
@pytest.mark.parametrize("n", [0, 1000, 256 * 320])
@pytest.mark.parametrize("stretch", [1.0, 2.5, 4.0])
@pytest.mark.parametrize("dtype", [F16, BF16])
@pytest.mark.parametrize("ch", [64, 128])
def test_span_conv_passes_of_a_group(n, stretch, dtype, ch):
    td = torch.float16 if dtype == F16 else torch.bfloat16
    g = torch.Generator(device="cuda").manual_seed(3)
    n_in = int(n * stretch) + 40
    x = torch.randn((n_in, ch), generator=g, device="cuda").to(td)
    w = (torch.randn((27, ch, ch), generator=g, device="cuda") * 0.1).to(td)
    o = (torch.arange(n, device="cuda") * stretch).long()
    nbr = torch.stack([o + 4 * (k // 3) + k % 3 for k in range(27)]) if n else torch.zeros((27, 0), dtype=torch.int64, device="cuda")
    nbr = torch.where(torch.rand(nbr.shape, generator=g, device="cuda") < 0.3, torch.full_like(nbr, -1), nbr)
    nbr[:, 5:6] = -1
    nbr[9:12] = -1                                              # a group without an entry
    cap = n + 7
    table = torch.zeros((27, cap), dtype=torch.int32, device="cuda")
    table[:, :n] = nbr.to(torch.int32)
    scale, shift = torch.rand(ch, generator=g, device="cuda") + 0.5, torch.randn(ch, generator=g, device="cuda")
    ctx = B.Context(16, 16, 64, n_slots=1)
    wp = torch.empty_like(w)
    ctx.pack_weights(dtype, w, wp)
    exp = torch.zeros((n, ch), device="cuda")
    for k in range(27):
        rows = (nbr[k] >= 0).nonzero().squeeze(1)
        exp[rows] += x[nbr[k][rows]].float() @ w[k].float()
    for epi in (EPI_NONE, EPI_AFFINE, EPI_AFFINE_RELU):
        y = torch.full((cap, ch), 77.0, dtype=td, device="cuda")
        aff = (None, None) if epi == EPI_NONE else (scale, shift)
        ctx.spconv(dtype, x, wp, *aff, epi, table, torch.tensor([n], dtype=torch.int32, device="cuda"), cap, y, w_layout=B.W_PACKED,
                   map_hint=B.SUBM)
        ctx.status_sync()
        want = exp if epi == EPI_NONE else exp * scale + shift
        want = want.clamp(min=0.0) if epi == EPI_AFFINE_RELU else want
        rms = float(want.square().mean().sqrt()) if n else 0.0
        tol = 2.0 ** -10 if dtype == F16 else 2.0 ** -7
        assert bool(((y[:n].float() - want).abs() <= tol * (want.abs() + rms)).all()), epi
        assert bool((y[n:] == 77.0).all())
    ctx.close()


def _stretched(n, stretch):
    """27 taps over n rows: row o reads about row o * stretch, three neighbouring rows at the taps of a group, so that a tile's
    interval is about `stretch` times its rows; a third of the entries absent, all of a row's and all of a group's too."""
    g = torch.Generator(device="cuda").manual_seed(7)
    o = (torch.arange(n, device="cuda") * stretch).long()
    nbr = torch.stack([o + 4 * (k // 3) + k % 3 for k in range(27)])
    nbr = torch.where(torch.rand(nbr.shape, generator=g, device="cuda") < 1 / 3, torch.full_like(nbr, -1), nbr)
    nbr[:, n // 2] = -1
    nbr[9:12] = -1
    return nbr.to(torch.int32).contiguous(), int(n * stretch) + 40


def _span_forms(nbr, n, cap, ch):
    """Forms (1, 2 or 3: passes) in which the span kernel runs the groups of this map, and the tile height it takes: its rule
    over the constants in its source."""
    src = open(os.path.join(os.path.dirname(B.__file__), "csrc", "spconv_span.hip")).read()
    cfg = re.search(r"struct SpanCfg<%d, %d> \{.*?\n\};" % (ch, ch), src, re.S).group(0)
    tr, mt0, mts = (int(v) for v in re.search(r"TR = (\d+), MT0 = (\d+), MTS = (\d+);", cfg).groups())
    first, nxt = ([int(v) for v in re.search(name + r"\[MTS\] = \{([^}]*)\}", cfg).group(1).split(",")] for name in ("kFirst", "kNext"))
    step = min(-(-(-(-cap // (64 * mt0))) // 8) * 8, 256) // 8
    cost = [first[i] + (-(-(-(-(-(-n // (64 * (mt0 + i)))) // 8)) // step) - 1) * nxt[i] for i in range(mts)]
    mt = mt0 + cost.index(min(cost))
    forms = set()
    t = nbr[:, :n].cpu().numpy().reshape(9, 3, n)
    for r0 in range(0, n, 64 * mt):
        split = r0 + 64 * ((mt + 1) // 2)
        for g in t[:, :, r0:r0 + 64 * mt]:
            lengths = []
            for part in (g, g[:, :split - r0], g[:, split - r0:]):
                e = part[part >= 0]
                lengths.append(int(e.max()) - int(e.min()) + 1 if e.size else 0)
            if lengths[0]:
                forms.add(1 if lengths[0] <= tr else 2 if max(lengths[1:]) <= tr else 3)
    return forms, mt


# A group's interval one row below, at and one beyond the row buffer (400 rows at 64 channels, 224 at 128): of a whole tile
# (one pass, else two), and of a tile's first half where the whole does not fit anyway (two passes, else three).  A tile of
# 192 rows at 64 channels, of 128 at 128 (16 385 rows and more).
@pytest.mark.parametrize("ch,rows,n,limit", [(64, 192, 192, 400), (128, 128, 16385, 224)])
@pytest.mark.parametrize("beyond", [-1, 0, 1])
@pytest.mark.parametrize("half", [False, True])
@pytest.mark.parametrize("dtype", [F16, BF16])
def test_span_conv_row_buffer_limit(ch, rows, n, limit, beyond, half, dtype):
    td = torch.float16 if dtype == F16 else torch.bfloat16
    part = 64 * ((rows // 64 + 1) // 2) if half else rows        # the rows that share the interval
    r = torch.arange(n, device="cuda") % rows
    at = torch.where(r < part, r * (limit + beyond - 3) // (part - 1), limit + 100 + r - part)
    at = at + (torch.arange(n, device="cuda") // rows * 640) % 20000
    nbr = torch.stack([at + k % 3 for k in range(27)])
    nbr[:, 7::11] = -1                                           # (neither of a tile's ends)
    nbr = nbr.to(torch.int32).contiguous()
    forms, mt = _span_forms(nbr, n, n, ch)
    assert 64 * mt == rows and (3 if half else 2) - (beyond <= 0) in forms
    n_in = int(nbr.max()) + 1
    g = torch.Generator(device="cuda").manual_seed(limit + beyond)
    x = torch.randn((n_in, ch), generator=g, device="cuda").to(td)
    w = (torch.randn((27, ch, ch), generator=g, device="cuda") * 0.1).to(td)
    ctx = B.Context(16, 16, 64, n_slots=1)
    wp = torch.empty_like(w)
    ctx.pack_weights(dtype, w, wp)
    got = []
    for hint in (B.SUBM, B.MAP_ANY):
        y = torch.empty((n, ch), dtype=td, device="cuda")
        ctx.spconv(dtype, x, wp, None, None, EPI_NONE, nbr, torch.tensor([n], dtype=torch.int32, device="cuda"), n, y,
                   w_layout=B.W_PACKED, map_hint=hint)
        ctx.status_sync()
        got.append(y)
    exp = torch.zeros((n, ch), device="cuda")
    for k in range(27):
        rs = (nbr[k] >= 0).nonzero().squeeze(1)
        exp[rs] += x[nbr[k][rs].long()].float() @ w[k].float()
    rms, tol = float(exp.square().mean().sqrt()), 2.0 ** -10 if dtype == F16 else 2.0 ** -7      # as in _check_conv
    assert bool(((got[0].float() - exp).abs() <= tol * (exp.abs() + rms)).all())
    assert torch.equal(got[0].view(torch.int16), got[1].view(torch.int16))
    ctx.close()


# The kernels of the hints add in one order: the same bits, whichever form a group takes (one pass, two halves, three taps)
@pytest.mark.parametrize("n,stretch,forms", [(2, 1.0, ({1}, {1})), (129, 1.0, ({1}, {1})), (1000, 4.0, ({3}, {3})), (16385, 2.5, ({2}, {2})),
                                             (81920, 1.0, ({1}, {1})), (81920, 1.5, ({2}, {2}))])
@pytest.mark.parametrize("dtype", [F16, BF16])
@pytest.mark.parametrize("ch", [64, 128])
def test_hint_never_changes_a_bit(n, stretch, forms, dtype, ch):
    td = torch.float16 if dtype == F16 else torch.bfloat16
    nbr, n_in = _stretched(n, stretch)
    assert _span_forms(nbr, n, n, ch)[0] >= forms[ch == 128]     # (a ragged last tile's may be another)
    g = torch.Generator(device="cuda").manual_seed(n + ch)
    x = torch.randn((n_in, ch), generator=g, device="cuda").to(td)
    w = (torch.randn((27, ch, ch), generator=g, device="cuda") * 0.1).to(td)
    ctx = B.Context(16, 16, 64, n_slots=1)
    wp = torch.empty_like(w)
    ctx.pack_weights(dtype, w, wp)
    got = []
    for hint, rows in ((B.SUBM, None), (B.MAP_ANY, None), (B.STRIDED, None), (B.MAP_ANY, 1 << 26)):    # the last: rows by address
        y = torch.empty((n, ch), dtype=td, device="cuda")
        ctx.spconv(dtype, x, wp, None, None, EPI_NONE, nbr, torch.tensor([n], dtype=torch.int32, device="cuda"), n, y,
                   w_layout=B.W_PACKED, map_hint=hint, n_in_rows=rows)
        ctx.status_sync()
        got.append(y.view(torch.int16))
    for other in got[1:]:
        assert torch.equal(got[0], other)
    ctx.close()


@pytest.mark.parametrize("n", [513, 40001, 70001, 131072 + 5000])
def test_span_conv_rounds_taps_outside_an_interval(n):
    _check_conv(n, 64, 64, B.SUBM, True)


# Blocks of 128 rows.  A capacity of up to 4 * 8 192 blocks gets a block for each tile, a row more 8 192 blocks that loop over
# the tiles there are: one tile for all but the last, one more than blocks, a second tile for half of those of every XCD.  64 channels of
# 2^25 rows and more (128 of 2^24) are read by address instead of through a descriptor.  Levels of this size leave groups out
# but for submanifold maps and 128 output channels, which walk straight over the taps.
@pytest.mark.parametrize("cin,cout,n,loop,hint", [
    (64, 64, 8192 * 128 - 129, True, B.MAP_ANY), (64, 64, 8192 * 128 + 1, True, B.MAP_ANY), (64, 64, 8192 * 128 + 77, True, B.STRIDED),
    (64, 64, 8192 * 128 * 3 // 2 + 77, True, B.MAP_ANY), (64, 64, 8192 * 128 * 3 // 2 + 77, False, B.MAP_ANY),
    (64, 128, 300, True, B.SUBM), (64, 128, 8192 * 128 - 129, True, B.MAP_ANY), (64, 128, 8192 * 128 + 1, True, B.SUBM),
    (64, 128, 8192 * 128 + 77, True, B.STRIDED), (64, 128, 8192 * 128 * 3 // 2 + 77, True, B.SUBM),
    (64, 128, 8192 * 128 * 3 // 2 + 77, False, B.MAP_ANY),
    (128, 128, 8192 * 128 + 77, True, B.MAP_ANY), (128, 128, 8192 * 128 * 3 // 2 + 77, True, B.MAP_ANY)])
def test_direct_conv_grid_limit(cin, cout, n, loop, hint):
    assert _kernel(cin, cout, hint) == "k_spconv_direct"
    cap = 4 * 8192 * 128 + (1 if loop else 0)
    _check_conv(n, cin, cout, hint, False, cap=cap)
    if loop:
        _check_conv(n, cin, cout, hint, False, cap=cap, rows_in=(1 << 25) + 3)


# Tiles of 32 rows to 256 blocks of 15 waves (12 by address), a block in a CU, whose waves take the block's tiles one by one: a tile, fewer tiles than
# blocks, as many, some of a block's waves with a tile, a tile less and more than all waves, many a wave; a capacity of the rows and of
# many times as many.  32 channels of 2^26 rows and more (64 of 2^25) are read by address.
@pytest.mark.parametrize("cin,cout", [(32, 64), (64, 32)])
@pytest.mark.parametrize("n", [1, 300, 255 * 32 + 1, 256 * 32 + 1, 256 * 5 * 32 + 1, 256 * 12 * 32 - 33, 256 * 12 * 32 + 1,
                               256 * 15 * 32 - 33, 256 * 15 * 32 + 1, 8192 * 128 - 129,
                               8192 * 128 * 3 // 2 + 77])
def test_resident_conv_grid_limit(cin, cout, n):
    for hint in (B.SUBM, B.STRIDED, B.MAP_ANY):
        assert _kernel(cin, cout, hint) == "k_spconv_direct_resident"
    _check_conv(n, cin, cout, B.MAP_ANY, False)
    _check_conv(n, cin, cout, B.SUBM, False, cap=4 * 8192 * 128 + 1)
    _check_conv(n, cin, cout, B.STRIDED, False, cap=n + 5, rows_in=((1 << 31) // cin) + 3)


# 32 -> 32 in a capacity of many times its grid, which loops over the tiles of 32 rows a wave there are
@pytest.mark.parametrize("n", [1, 8192 * 256 + 300])
def test_narrow_conv_grid_limit(n):
    assert _kernel(32, 32, B.MAP_ANY) == "k_spconv_narrow"
    _check_conv(n, 32, 32, B.MAP_ANY, False, cap=4 * 8192 * 256 + 1)


# Blocks of 256 rows; those beyond the count leave at once.  No row, the edges of a wave and of a block, a count above the capacity
@pytest.mark.parametrize("dt", [torch.float16, torch.bfloat16])
@pytest.mark.parametrize("cin,cout", [(4, 16), (4, 32), (16, 16)])
@pytest.mark.parametrize("n,cap", [(0, 1), (0, 300), (1, 1), (63, 70000), (64, 64), (255, 256), (256, 70000), (257, 70000), (1025, 1100), (600, 513)])
def test_rows_conv_few_rows_of_a_capacity(n, cap, cin, cout, dt):
    """Small whole numbers: every fp32 sum is exact in any order, and both 16-bit types hold it."""
    rows, n_in = min(n, cap), 400
    g = torch.Generator(device="cuda").manual_seed(n + cin + cout)
    x = torch.randint(-1, 2, (n_in, cin), generator=g, device="cuda").to(dt)
    w = torch.randint(-1, 2, (27, cin, cout), generator=g, device="cuda").to(dt)
    nbr = torch.full((27, cap), 1 << 30, dtype=torch.int32, device="cuda")       # beyond the rows: entries that would be reported
    nbr[:, :rows] = torch.randint(-n_in, n_in, (27, rows), generator=g, device="cuda").clamp_(min=-1).to(torch.int32)
    exp = torch.zeros((rows, cout), device="cuda")
    for k in range(27):
        at = (nbr[k][:rows] >= 0).nonzero().squeeze(1)
        exp[at] += x[nbr[k][at].long()].float() @ w[k].float()
    assert rows == 0 or float(exp.abs().max()) <= 254
    y = torch.full((cap, cout), 77.0, dtype=dt, device="cuda")
    ctx = B.Context(16, 16, 64, n_slots=1)
    scale, shift = torch.full((cout,), 0.5, device="cuda"), torch.full((cout,), 1.0, device="cuda")
    ctx.spconv(F16 if dt == torch.float16 else BF16, x, w, scale, shift, EPI_AFFINE_RELU, nbr, torch.tensor([n], dtype=torch.int32, device="cuda"),
               cap, y)
    ctx.status_sync()
    assert torch.equal(y[:rows].float(), (exp * 0.5 + 1.0).clamp_(min=0.0).to(dt).float()) and bool((y[rows:] == 77.0).all())
    ctx.close()


def _kernel(cin, cout, hint):
    ctx = B.Context(16, 16, 64, n_slots=1)
    name = ctx.spconv_kernel(F16, cin, cout, hint)
    ctx.close()
    return name


# Blocks of 128 rows that have entries in no group, in one, in every one, and whose waves differ; the last block ragged.  At 64 -> 64 up to
# 256 blocks walk straight over the taps, more of them leave groups out, in a loop over the tiles where the capacity is large; at
# 32 -> 64 and 64 -> 32 each wave leaves out the groups its own rows do not have.
@pytest.mark.parametrize("cin,cout", [(32, 64), (64, 32), (64, 64)])
@pytest.mark.parametrize("n,cap", [(1, 1), (128, 128), (129, 129), (1000, 1000), (33000, 33000), (66000, 66000), (8192 * 128 + 300, 4 * 8192 * 128 + 1)])
def test_direct_conv_groups_without_entries(cin, cout, n, cap):
    g = torch.Generator(device="cuda").manual_seed(cin + cout + n)
    n_in = 500
    x = torch.randn((n_in, cin), generator=g, device="cuda").half()
    w = (torch.randn((27, cin, cout), generator=g, device="cuda") * 0.1).half()
    nbr = torch.randint(0, n_in, (27, n), generator=g, device="cuda")
    group, block, wave = torch.arange(27, device="cuda") // 3, torch.arange(n, device="cuda") // 128, torch.arange(n, device="cuda") // 32
    keep = (block % 4 == 1)[None, :] & (group[:, None] == block[None, :] % 9) | (block % 4 == 2)[None, :] | \
        (block % 4 == 3)[None, :] & (group[:, None] == wave[None, :] % 9)      # blocks 0, 4, ..: nothing
    nbr = torch.where(keep & (torch.rand((27, n), generator=g, device="cuda") < 0.7), nbr, torch.full_like(nbr, -1)).to(torch.int32)
    table = torch.zeros((27, cap), dtype=torch.int32, device="cuda")
    table[:, :n] = nbr
    exp = torch.zeros((n, cout), device="cuda")
    for k in range(27):
        rows = (nbr[k] >= 0).nonzero().squeeze(1)
        exp[rows] += x[nbr[k][rows].long()].float() @ w[k].float()
    rms = float(exp.square().mean().sqrt())
    ctx = B.Context(16, 16, 64, n_slots=1)
    wp = torch.empty_like(w)
    ctx.pack_weights(F16, w, wp)
    got = []
    for hint in (B.MAP_ANY, B.STRIDED, B.SUBM):
        y = torch.full((cap + 2, cout), 77.0, dtype=torch.float16, device="cuda")
        ctx.spconv(F16, x, wp, None, None, EPI_NONE, table, torch.tensor([n], dtype=torch.int32, device="cuda"), cap, y[:cap],
                   w_layout=B.W_PACKED, map_hint=hint)
        ctx.status_sync()
        assert float(((y[:n].float() - exp).abs() - 2.0 ** -10 * (exp.abs() + rms)).max()) <= 0.0     # as in _check_conv
        assert bool((y[n:] == 77.0).all())
        got.append(y)
    assert torch.equal(got[0], got[1]) and torch.equal(got[0], got[2])         # the hint chooses a way, never a result
    ctx.close()


# 64 -> 64: levels of up to 256 blocks walk straight over the taps, larger ones leave out the groups no row of a block has, submanifold
# ones never: the same bits on both sides of the line.  (32 -> 64 and 64 -> 32 take one way at all sizes and hints.)
@pytest.mark.parametrize("cin,cout,line", [(32, 64, 512 * 128), (64, 32, 256 * 128), (64, 64, 256 * 128)])
@pytest.mark.parametrize("beyond", [0, 1])
def test_direct_conv_straight_and_leaving_out(cin, cout, line, beyond):
    n = line + beyond
    g = torch.Generator(device="cuda").manual_seed(cin + cout)
    n_in = 5000
    x = torch.randn((n_in, cin), generator=g, device="cuda").half()
    w = (torch.randn((27, cin, cout), generator=g, device="cuda") * 0.1).half()
    nbr = torch.randint(0, n_in, (27, n), generator=g, device="cuda")
    block = torch.arange(n, device="cuda") // 128
    keep = (torch.arange(27, device="cuda")[:, None] // 3 + block[None, :]) % 4 == 0          # two or three groups of a block
    keep &= torch.rand((27, n), generator=g, device="cuda") < 0.7
    nbr = torch.where(keep, nbr, torch.full_like(nbr, -1)).to(torch.int32).contiguous()
    ctx = B.Context(16, 16, 64, n_slots=1)
    wp = torch.empty_like(w)
    ctx.pack_weights(F16, w, wp)
    got = []
    for hint in (B.MAP_ANY, B.SUBM):
        y = torch.empty((n, cout), dtype=torch.float16, device="cuda")
        ctx.spconv(F16, x, wp, None, None, EPI_NONE, nbr, torch.tensor([n], dtype=torch.int32, device="cuda"), n, y,
                   w_layout=B.W_PACKED, map_hint=hint)
        ctx.status_sync()
        got.append(y)
    exp = torch.zeros((n, cout), device="cuda")
    for k in range(27):
        rows = (nbr[k] >= 0).nonzero().squeeze(1)
        exp[rows] += x[nbr[k][rows].long()].float() @ w[k].float()
    rms = float(exp.square().mean().sqrt())
    assert float(((got[0].float() - exp).abs() - 2.0 ** -10 * (exp.abs() + rms)).max()) <= 0.0     # as in _check_conv
    assert torch.equal(got[0], got[1])
    ctx.close()


# inputs of less than 4 GiB are read through a buffer descriptor, larger ones by address; any negative entry is absent
@pytest.mark.parametrize("cin,cout,n_in", [(64, 32, 1 << 10), (64, 64, (1 << 25) - 1), (64, 64, 1 << 25), (32, 32, (1 << 25) + 3),
                                           (128, 128, (1 << 24) - 1)])
def test_direct_conv_input_sizes_and_negative_entries(cin, cout, n_in):
    n = 300
    g = torch.Generator(device="cuda").manual_seed(n_in)
    x = torch.randn((n_in, cin), generator=g, device="cuda", dtype=torch.float16)
    w = (torch.randn((27, cin, cout), generator=g, device="cuda") * 0.1).half()
    nbr = torch.randint(0, n_in, (27, n), generator=g, device="cuda")
    nbr[:, ::7] = n_in - 1                                     # the last row
    absent = torch.tensor([-1, -2, -3, -(1 << 24), -(1 << 25) + 1, -(1 << 31) + 1, -(1 << 31)], device="cuda")
    drop = torch.rand((27, n), generator=g, device="cuda") < 0.5
    nbr = torch.where(drop, absent[torch.randint(0, 7, (27, n), generator=g, device="cuda")], nbr).to(torch.int32).contiguous()
    ctx = B.Context(16, 16, 64, n_slots=1)
    wp = torch.empty_like(w)
    ctx.pack_weights(F16, w, wp)
    y = torch.empty((n, cout), dtype=torch.float16, device="cuda")
    ctx.spconv(F16, x, wp, None, None, EPI_NONE, nbr, torch.tensor([n], dtype=torch.int32, device="cuda"), n, y, w_layout=B.W_PACKED)
    ctx.status_sync()
    exp = torch.zeros((n, cout), device="cuda")
    for k in range(27):
        rows = (~drop[k]).nonzero().squeeze(1)
        exp[rows] += x[nbr[k][rows].long()].float() @ w[k].float()
    rms = float(exp.square().mean().sqrt())
    assert float(((y.float() - exp).abs() - 2.0 ** -10 * (exp.abs() + rms)).max()) <= 0.0
    ctx.close()


@pytest.mark.parametrize("cin", [64, 128])
def test_quantised_conv_addressing_and_negative_entries(cin):
    """Rows by buffer descriptor and (more rows vouched for than 4 GiB hold) by address: the same integers, exactly."""
    n, n_in, cout = 300, 5000, 64
    g = torch.Generator(device="cuda").manual_seed(cin)
    x = torch.randint(-127, 128, (n_in, cin), generator=g, device="cuda").to(torch.int8)
    w = torch.randint(-3, 4, (27, cin, cout), generator=g, device="cuda").to(torch.int8)
    nbr = torch.randint(0, n_in, (27, n), generator=g, device="cuda")
    nbr[:, ::7] = n_in - 1
    absent = torch.tensor([-1, -2, -(1 << 25), -(1 << 26) + 1, -(1 << 31)], device="cuda")
    drop = torch.rand((27, n), generator=g, device="cuda") < 0.5
    nbr = torch.where(drop, absent[torch.randint(0, 5, (27, n), generator=g, device="cuda")], nbr).to(torch.int32).contiguous()
    exp = torch.zeros((n, cout), device="cuda", dtype=torch.float64)
    for k in range(27):
        rows = (~drop[k]).nonzero().squeeze(1)
        exp[rows] += x[nbr[k][rows].long()].double() @ w[k].double()
    ctx = B.Context(16, 16, 64, n_slots=1)
    wp = torch.empty((27 * cin * cout,), dtype=torch.int8, device="cuda")
    ctx.pack_weights_i8(w, wp)
    mul, add = torch.full((cout,), 2.0 ** -8, device="cuda"), torch.zeros(cout, device="cuda")
    want = (exp * 2.0 ** -8).float().half()                      # sums below 2^24: exact until the one rounding to fp16
    for rows_in in (n_in, 1 << 27):
        y = torch.empty((n, cout), dtype=torch.float16, device="cuda")
        ctx.spconv_i8(x, wp, cin, cout, mul, add, False, nbr, torch.tensor([n], dtype=torch.int32, device="cuda"), n, y,
                      n_in_rows=rows_in)
        ctx.status_sync()
        assert torch.equal(y, want)
    ctx.close()


# around a wave's 32 rows, a block's 128 or 256, and the rows of all resident blocks (131 072); more rows vouched for than 4 GiB hold
@pytest.mark.parametrize("dt", [torch.float16, torch.bfloat16])
@pytest.mark.parametrize("cin", [16, 32])
@pytest.mark.parametrize("n,rows_in", [(0, None), (1, None), (31, None), (32, 1 << 28), (33, None), (127, None), (129, None), (255, None),
                                       (257, 1 << 28), (131072, None), (131073, None), (262144 + 4001, None)])
def test_narrow_conv_row_counts(n, rows_in, cin, dt):
    """Small whole numbers: every fp32 sum is exact in any order, and both 16-bit types hold it."""
    n_in, cout, cap = 4000, 32, n + 7
    g = torch.Generator(device="cuda").manual_seed(n + cin)
    x = torch.randint(-1, 2, (n_in, cin), generator=g, device="cuda").to(dt)
    w = torch.randint(-1, 2, (27, cin, cout), generator=g, device="cuda").to(dt)
    nbr = torch.randint(-n_in, n_in, (27, cap), generator=g, device="cuda")
    nbr = torch.where(nbr < 0, torch.where(nbr % 3 == 0, nbr * 100000, -1), nbr).to(torch.int32).contiguous()
    ctx = B.Context(16, 16, 64, n_slots=1)
    edt = F16 if dt == torch.float16 else BF16
    wp = torch.empty_like(w)
    ctx.pack_weights(edt, w, wp)
    y = torch.full((cap, cout), 77.0, dtype=dt, device="cuda")
    scale, shift = torch.full((cout,), 0.5, device="cuda"), torch.full((cout,), 1.0, device="cuda")
    ctx.spconv(edt, x, wp, scale, shift, EPI_AFFINE_RELU, nbr, torch.tensor([n], dtype=torch.int32, device="cuda"), cap, y,
               w_layout=B.W_PACKED, n_in_rows=rows_in)
    ctx.status_sync()
    exp = torch.zeros((n, cout), device="cuda")
    for k in range(27):
        rows = (nbr[k][:n] >= 0).nonzero().squeeze(1)
        exp[rows] += x[nbr[k][rows].long()].float() @ w[k].float()
    assert n == 0 or float(exp.abs().max()) <= 254               # half of it and one: at most 128, a half at the least step
    want = (exp * 0.5 + 1.0).clamp_(min=0.0)
    assert torch.equal(y[:n].float(), want.to(dt).float()) and bool((y[n:] == 77.0).all())
    ctx.close()


@pytest.mark.parametrize("e4m3", [False, True])
@pytest.mark.parametrize("cin,cout", [(64, 64), (128, 32)])
@pytest.mark.parametrize("n", [1, 15, 16, 17, 31, 32, 33, 127, 128, 129, 1025])
def test_quantised_conv_row_counts(n, cin, cout, e4m3):
    """Row counts at the edges of a tile (16), a wave (32) and a block (128)."""
    _check_quantised(n, n + 5, cin, cout, e4m3)


# Tiles of 32 rows, taken by the waves of up to 256 blocks.  128 -> 64: 32 rows a wave of levels of up to 98 304 rows; larger ones in int8
# run whole steps of 65 536 rows with 64 a wave, the rest too if it is half a step, else with 32; the grid holds the tiles, whatever the
# capacity: both sides of each line, rests of a row, a tile and just under half a step, and few rows of a large capacity.
@pytest.mark.parametrize("e4m3", [False, True])
@pytest.mark.parametrize("cin,cout", [(64, 32), (64, 64), (128, 32), (128, 64)])
@pytest.mark.parametrize("n,cap", [(98304, 98304), (98304, 98305), (98305, 98305), (131072, 131072), (131073, 131073), (131072 + 129, 300000),
                                   (300, 200000), (98200, 400000), (163839, 163839), (163840, 200000), (196608, 196609),
                                   (196608 + 32767, 196608 + 32767), (5 * 65536 + 1025, 5 * 65536 + 1025), (9 * 65536 - 1, 700000)])
def test_quantised_conv_rows_a_wave(n, cap, cin, cout, e4m3):
    _check_quantised(n, cap, cin, cout, e4m3)


# Rows by buffer descriptor and (more rows vouched for than 4 GiB hold) by address, in every form of the kernels: shapes, operands, results.
# Part of a tile, a tile and a row, a tile for every wave of 12 and of 15 in 256 blocks and a row more
@pytest.mark.parametrize("n", [5, 33, 256 * 12 * 32 + 1, 256 * 15 * 32 + 1])
@pytest.mark.parametrize("cin,cout", [(64, 32), (64, 64), (128, 32), (128, 64)])
@pytest.mark.parametrize("e4m3,out", [(False, torch.float16), (False, torch.int8), (True, torch.float16), (True, torch.float32)])
def test_quantised_conv_by_descriptor_and_by_address(e4m3, out, cin, cout, n):
    """Small whole numbers: the sums, halved and clamped as the call says, are exact in every type."""
    n_in, cap = 3000, n + 3
    g = torch.Generator(device="cuda").manual_seed(n + cin + cout)
    xv, wv = torch.randint(-2, 3, (n_in, cin), generator=g, device="cuda"), torch.randint(-1, 2, (27, cin, cout), generator=g, device="cuda")
    nbr = torch.randint(-n_in, n_in, (27, cap), generator=g, device="cuda")
    nbr = torch.where(nbr < 0, torch.where(nbr % 3 == 0, nbr * 500000, -1), nbr).to(torch.int32).contiguous()
    exp = torch.zeros((n, cout), device="cuda")
    for k in range(27):
        at = (nbr[k, :n] >= 0).nonzero().squeeze(1)
        exp[at] += xv[nbr[k, at].long()].float() @ wv[k].float()
    ctx = B.Context(16, 16, 64, n_slots=1)
    x, w = xv.to(torch.int8), wv.to(torch.int8)
    if e4m3:
        x, w = torch.empty((n_in, cin), dtype=torch.uint8, device="cuda"), torch.empty((27, cin, cout), dtype=torch.uint8, device="cuda")
        ctx.quantize_e4m3(xv.float(), 1.0, x)
        ctx.quantize_e4m3(wv.float(), 1.0, w)
    wp = torch.empty((27 * cin * cout,), dtype=torch.int8, device="cuda")
    ctx.pack_weights_i8(w.view(torch.int8), wp)
    mul, add = torch.full((cout,), 0.5, device="cuda"), torch.arange(cout, device="cuda").float() - 9.0
    want = (exp * 0.5 + add).clamp_(min=0.0)
    assert float(exp.abs().max()) <= 1024
    want = (want * 0.125).round().clamp_(max=127.0).to(torch.int8) if out == torch.int8 else want.to(out)
    count = torch.tensor([n], dtype=torch.int32, device="cuda")
    for rows_in in (n_in, (1 << 32) // cin + 3):
        y = torch.full((cap, cout), 77, dtype=out, device="cuda")
        if e4m3:
            ctx.spconv_e4m3(x, wp, cin, cout, mul, add, True, nbr, count, cap, y, n_in_rows=rows_in)
        elif out == torch.int8:
            ctx.spconv_i8(x, wp, cin, cout, mul, add, True, nbr, count, cap, y, inv_out_scale=0.125, n_in_rows=rows_in)
        else:
            ctx.spconv_i8(x, wp, cin, cout, mul, add, True, nbr, count, cap, y, n_in_rows=rows_in)
        ctx.status_sync()
        assert torch.equal(y[:n], want) and bool((y[n:] == 77).all())
    ctx.close()


# A capacity of many times the rows; and the rows of thousands of blocks
@pytest.mark.parametrize("cin,cout,e4m3", [(128, 32, False), (64, 64, True), (128, 32, True), (128, 64, True), (64, 64, False)])
@pytest.mark.parametrize("n", [300, 8192 * 128 + 77])
def test_quantised_conv_large_capacity(n, cin, cout, e4m3):
    _check_quantised(n, 4 * 8192 * 128, cin, cout, e4m3)


def _check_quantised(n, cap, cin, cout, e4m3):
    """n rows of `cap`.  Small whole numbers, so both types are exact."""
    n_in = 300
    g = torch.Generator(device="cuda").manual_seed(n + cin)
    xv = torch.randint(-2, 3, (n_in, cin), generator=g, device="cuda")
    wv = torch.randint(-1, 2, (27, cin, cout), generator=g, device="cuda")
    nbr = torch.randint(-n_in, n_in, (27, cap), generator=g, device="cuda").clamp_(min=-1).to(torch.int32)
    exp = torch.zeros((n, cout), device="cuda", dtype=torch.float64)
    for k in range(27):
        j = nbr[k, :n].long()
        exp += torch.where((j >= 0)[:, None], xv[j.clamp(min=0)].double() @ wv[k].double(), 0.0)
    ctx = B.Context(16, 16, 64, n_slots=1)
    if e4m3:
        x = torch.empty((n_in, cin), dtype=torch.uint8, device="cuda")
        w = torch.empty((27, cin, cout), dtype=torch.uint8, device="cuda")
        ctx.quantize_e4m3(xv.float(), 1.0, x)
        ctx.quantize_e4m3(wv.float(), 1.0, w)
    else:
        x, w = xv.to(torch.int8), wv.to(torch.int8)
    wp = torch.empty((27 * cin * cout,), dtype=torch.int8, device="cuda")
    ctx.pack_weights_i8(w.view(torch.int8), wp)
    one, zero = torch.ones(cout, device="cuda"), torch.zeros(cout, device="cuda")
    y = torch.full((cap, cout), 7.0, dtype=torch.float16, device="cuda")
    call = ctx.spconv_e4m3 if e4m3 else ctx.spconv_i8
    call(x, wp, cin, cout, one, zero, False, nbr, torch.tensor([n], dtype=torch.int32, device="cuda"), cap, y, n_in_rows=n_in)
    ctx.status_sync()
    assert exp.abs().max() <= 2048                               # every sum is a whole number that fp16 holds
    assert torch.equal(y[:n].double(), exp) and bool((y[n:] == 7.0).all())
    ctx.close()


@pytest.mark.parametrize("dt", [np.float32, np.float16])
@pytest.mark.parametrize("n,off", [(1, 0), (7, 0), (8, 0), (9, 0), (2048, 0), (2055, 0), (5000, 1), (5000, 4)])
def test_quantisers_tails_and_alignment(n, off, dt):
    x = np.random.RandomState(n).normal(0, 40, n).astype(dt)
    ctx = B.Context(16, 16, 64, n_slots=1)
    buf = torch.zeros(n + off, dtype=torch.float32 if dt == np.float32 else torch.float16, device="cuda")
    buf[off:] = torch.from_numpy(x).cuda()
    for call, ref, td in ((ctx.quantize_i8, oracle.quantize_i8, torch.int8), (ctx.quantize_e4m3, oracle.quantize_e4m3, torch.uint8)):
        q = torch.full((off + n + 9,), 99, dtype=td, device="cuda")
        call(buf[off:], 1.5, q[off:off + n])
        assert np.array_equal(q[off:off + n].cpu().numpy(), ref(x.astype(np.float32), 1.5))
        assert q[off + n:].tolist() == [99] * 9 and q[:off].tolist() == [99] * off
    ctx.close()


# cells shared by 1 .. 70 points, waves that end in the middle
@pytest.mark.parametrize("n,side", [(1, 4), (63, 1), (64, 4), (65, 4), (300, 1), (1000, 8), (1000, 64)])
def test_voxelize_first_points(n, side):
    rng = np.random.RandomState(n + side)
    pts = np.concatenate([rng.uniform(0, side, (n, 3)), rng.uniform(0, 1, (n, 1))], 1).astype(np.float32)
    pts[::13, 0] = -1.0
    grid = (side, side, side)
    spec = VoxelSpec((0.0, 0.0, 0.0), (1.0, 1.0, 1.0), grid)
    ctx = B.Context(n, n, cells_of(grid, 1), n_slots=1)
    i32 = dict(dtype=torch.int32, device="cuda")
    coords, feats, counts, nv = torch.zeros((n, 4), **i32), torch.full((n, 4), 5.0, device="cuda"), torch.full((n,), 5, **i32), torch.zeros(1, **i32)
    for _ in range(2):                                   # the second pass starts from the first one's buffers
        ctx.voxelize(torch.from_numpy(pts).cuda(), None, spec, n, coords, feats, counts, nv, index_slot=0)
    ctx.status_sync()
    oc, om, on = oracle.voxelize(pts, None, spec.lo, spec.vs, grid)
    v = len(oc)
    assert int(nv.item()) == v
    assert np.array_equal(coords[:v].cpu().numpy(), oc) and np.array_equal(counts[:v].cpu().numpy(), on)
    # sums of up to n fp32 values in another order: n * 2^-24 relative to the sum of magnitudes, at most side * count
    assert np.all(np.abs(feats[:v].cpu().numpy() - om) <= (n + 2) * 2.0 ** -24 * max(side, 1))
    assert not feats[v:].any() and not counts[v:].any()
    ctx.close()


def test_index_scan_of_more_than_16384_tiles():
    grid, nb, n = (1408, 1600, 40), 13, 20000            # 17 875 tiles of 65 536 cells
    rng = np.random.RandomState(5)
    pts = np.concatenate([rng.uniform(0, 1, (n, 3)) * np.array(grid), rng.uniform(0, 1, (n, 1))], 1).astype(np.float32)
    batch = rng.randint(0, nb, n).astype(np.int32)
    spec = VoxelSpec((0.0, 0.0, 0.0), (1.0, 1.0, 1.0), grid, n_batch=nb)
    ctx = B.Context(n, n, cells_of(grid, nb), n_slots=1)
    i32 = dict(dtype=torch.int32, device="cuda")
    coords, feats, counts, nv = torch.zeros((n, 4), **i32), torch.zeros((n, 4), device="cuda"), torch.zeros((n,), **i32), torch.zeros(1, **i32)
    ctx.voxelize(torch.from_numpy(pts).cuda(), torch.from_numpy(batch).cuda(), spec, n, coords, feats, counts, nv, index_slot=0)
    ctx.status_sync()
    oc, _, on = oracle.voxelize(pts, batch, spec.lo, spec.vs, grid, n_batch=nb)
    v = len(oc)
    assert int(nv.item()) == v and np.array_equal(coords[:v].cpu().numpy(), oc) and np.array_equal(counts[:v].cpu().numpy(), on)
    ctx.close()


def _sites(n, grid, seed):
    """n sites of a one-frame grid in key order."""
    g = torch.Generator().manual_seed(seed)
    k = torch.randperm(grid[0] * grid[1] * grid[2], generator=g)[:n].sort().values
    c = torch.stack([torch.zeros_like(k), k // (grid[0] * grid[1]), k // grid[0] % grid[1], k % grid[0]], 1)
    return k.cuda(), c.to(torch.int32).contiguous().cuda()


# 64 half-precision channels are 8 pieces of 16 bytes or, off a 16-byte address, 32 of 4; a step is 4096 x 256 pieces
@pytest.mark.parametrize("n,off", [(131072, 0), (131073, 0), (150001, 0), (32768, 2), (32769, 2), (70001, 2)])
def test_bev_flatten_steps_and_alignment(n, off):
    grid, c = (64, 64, 40), 64
    ctx = B.Context(16, 16, 64, n_slots=1)
    _, coords = _sites(n, grid, n)
    flat = torch.randn(n * c + off, device="cuda").half()
    feats = flat[off:].view(n, c)
    out = torch.full((1, grid[1], grid[0], grid[2] * c), 9.0, dtype=torch.float16, device="cuda")
    ctx.bev_flatten(F16, coords, feats, torch.tensor([n], dtype=torch.int32, device="cuda"), n, grid, 1, out)
    want = torch.zeros((grid[1], grid[0], grid[2], c), dtype=torch.float16, device="cuda")
    z, y, x = coords[:, 1].long(), coords[:, 2].long(), coords[:, 3].long()
    want[y, x, z] = feats
    assert torch.equal(out.view_as(want), want)
    ctx.close()


@pytest.mark.parametrize("nl,ni", [(40000, 40000), (90000, 70001)])
def test_fuse_rows_beyond_one_step(nl, ni):
    grid, cl, ci = (64, 64, 40), 32, 64                       # 12 pieces a row
    ctx = B.Context(16, nl + ni, cells_of(grid, 1), n_slots=1)
    (kl, lc), (ki, ic) = _sites(nl, grid, nl), _sites(ni, grid, ni + 1)
    lf, fi = torch.randn((nl, cl), device="cuda").half(), torch.randn((ni, ci), device="cuda").half()
    i32 = dict(dtype=torch.int32, device="cuda")
    co, fo, n = torch.zeros((nl + ni, 4), **i32), torch.full((nl + ni, cl + ci), 9.0, dtype=torch.float16, device="cuda"), torch.zeros(1, **i32)
    ctx.fuse(F16, lc, lf, torch.tensor([nl], **i32), nl, ic, fi, torch.tensor([ni], **i32), ni, grid, 1, nl + ni, co, fo, n)
    keys = torch.unique(torch.cat([kl, ki]))
    want = torch.zeros((len(keys), cl + ci), dtype=torch.float16, device="cuda")
    want[torch.searchsorted(keys, kl), :cl] = lf
    want[torch.searchsorted(keys, ki), cl:] = fi
    assert int(n.item()) == len(keys) and torch.equal(fo[:len(keys)], want) and bool((fo[len(keys):] == 9.0).all())
    ctx.close()
