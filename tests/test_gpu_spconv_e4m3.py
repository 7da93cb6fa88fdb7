"""GPU parity of the E4M3 quantiser (bit-exact) and the E4M3 sparse conv (exact products, fp32 accumulation on the
matrix cores against the oracle's exact accumulation: within fp32 summation error) through the C-ABI."""
import numpy as np
import pytest
import torch

import oracle
from helpers import assert_features_close, progress, worst_feature_ratio
from paper_2507_04123_amd import binding as B
from paper_2507_04123_amd import gen
from paper_2507_04123_amd.configs import get_config, SUBM, STRIDED
from paper_2507_04123_amd.pipeline import BranchRunner, cells_of, default_capacities, device_params

pytestmark = pytest.mark.gpu

# The products are exact, but the matrix cores do not add the 32 products of an instruction the way a chain of fp32
# additions would: they align them to the largest and drop low bits, so the result differs from the exactly
# accumulated one by up to a few 1e-4 of (|o| + rms(o)) when the operands span the format's whole range (measured
# worst 2.9e-4), and not at all when every partial sum is a small integer (test below).  Bar: 1e-3 for fp32 output,
# 2e-3 with the additional rounding to fp16.
RTOL_F32, RTOL_F16 = 1e-3, 2e-3


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _rand_sites(seed, grid, nb, n):
    gx, gy, gz = grid
    total = gx * gy * gz * nb
    keys = np.unique((gen.Stream(seed, 3).bits(3 * n) % np.uint64(total)).astype(np.int64))[:n]
    keys.sort()
    x = keys % gx; y = (keys // gx) % gy; z = (keys // (gx * gy)) % gz; b = keys // (gx * gy * gz)
    return np.stack([b, z, y, x], axis=1).astype(np.int32)


def _rand_codes(seed, shape, top=0x77):
    """Random finite codes of both signs, magnitudes up to code `top` (0x77 = 240), subnormals and zeros included."""
    b = gen.Stream(seed, 23).bits(2 * int(np.prod(shape))).reshape(2, -1)
    mag = (b[0] % np.uint64(top + 1)).astype(np.uint8)
    sign = ((b[1] & np.uint64(1)) << np.uint64(7)).astype(np.uint8)
    c = (mag | sign).reshape(shape)
    return np.where(c == 0x80, 0, c).astype(np.uint8)


def test_quantize_e4m3_bit_exact():
    ctx = B.Context(16, 16, 64, n_slots=1)
    st = gen.Stream(12, 1)
    special = np.array([0.0, -0.0, 1.0, -1.0, 1.0625, 1.1875, 448.0, 449.0, 463.9, 464.0, 480.0, 1e9, -1e9, np.inf, -np.inf, np.nan,
                        2.0 ** -10, 2.0 ** -10 * 1.0001, 2.0 ** -9, 2.0 ** -6, 2.0 ** -6 * 0.999, 7.5 * 2.0 ** -9, -7.5 * 2.0 ** -9],
                       np.float32)
    x = np.concatenate([special, st.normal(100000, 40.0).astype(np.float32), st.normal(50000, 0.01).astype(np.float32),
                        st.normal(50000, 300.0).astype(np.float32)])
    for inv in (1.0, 0.37, 3.0):
        q = torch.zeros(len(x), dtype=torch.uint8, device="cuda")
        ctx.quantize_e4m3(dev(x), inv, q)
        torch.cuda.synchronize()
        exp = oracle.quantize_e4m3(x, inv)
        assert np.array_equal(q.cpu().numpy(), exp), f"inv_scale {inv}"
        assert set(np.unique(exp)) >= {0x00, 0x7E, 0xFE}
    xh = x[np.isfinite(x) & (np.abs(x) < 6e4)].astype(np.float16)
    q = torch.zeros(len(xh), dtype=torch.uint8, device="cuda")
    ctx.quantize_e4m3(dev(xh), 0.5, q)
    assert np.array_equal(q.cpu().numpy(), oracle.quantize_e4m3(xh.astype(np.float32), 0.5))
    ctx.close()


@pytest.mark.parametrize("inv", [1.0, 2.0 ** -8, 0.37])
def test_quantize_e4m3_every_half(inv):
    """All 65 536 fp16 values, eight a thread: subnormal codes, ties, saturation, both zeros, infinities and numbers that are none."""
    x = np.arange(65536, dtype=np.uint16).view(np.float16)
    ctx = B.Context(16, 16, 64, n_slots=1)
    q = torch.empty(len(x), dtype=torch.uint8, device="cuda")
    ctx.quantize_e4m3(dev(x), inv, q)
    assert np.array_equal(q.cpu().numpy(), oracle.quantize_e4m3(x.astype(np.float32), inv))
    ctx.close()


def _check_conv(ctx, xq, wq, mul, add, relu, nbr_np, cap):
    n_out = nbr_np.shape[1]
    cin, cout = wq.shape[1], wq.shape[2]
    nbr = torch.full((27, cap), -1, dtype=torch.int32, device="cuda")
    nbr[:, :n_out] = dev(nbr_np)
    n_t = torch.tensor([n_out], dtype=torch.int32, device="cuda")
    wp = torch.empty((27 * cin * cout,), dtype=torch.int8, device="cuda")
    ctx.pack_weights_i8(dev(wq.view(np.int8)), wp)                     # a byte permutation: the codes travel as bytes
    exp = oracle.spconv_e4m3(xq, wq, mul, add, relu, nbr_np)
    d_x = dev(xq) if len(xq) else torch.zeros((1, cin), dtype=torch.uint8, device="cuda")
    for out_dtype, rtol in ((torch.float32, RTOL_F32), (torch.float16, RTOL_F16)):
        out = torch.full((cap, cout), 55.0, dtype=out_dtype, device="cuda")
        ctx.spconv_e4m3(d_x, wp, cin, cout, dev(mul), dev(add), relu, nbr, n_t, cap, out)
        torch.cuda.synchronize()
        ctx.status_sync()
        got = out[:n_out].float().cpu().numpy()
        progress(f"spconv_e4m3 {cin}->{cout} n_out={n_out} relu={relu} out={out_dtype}: worst ratio {worst_feature_ratio(got, exp):.2e}")
        assert_features_close(got, exp, rtol, f"e4m3 conv {cin}->{cout} {out_dtype}")
        if n_out < cap:
            assert int((out[n_out:] != 55.0).sum().item()) == 0
    return exp


@pytest.mark.parametrize("cin,cout", [(64, 64), (64, 32), (128, 64), (128, 32)])
def test_spconv_e4m3_random_maps(cin, cout):
    ctx = B.Context(16, 4096, 64 * 64 * 8, n_slots=1)
    st = gen.Stream(cin + cout, 19)
    grid, nb = (14, 11, 6), 2
    coords = _rand_sites(cin * 3 + cout, grid, nb, 1100)
    xq = _rand_codes(cin, (len(coords), cin))
    wq = _rand_codes(cout, (27, cin, cout), top=0x47)                    # weights up to 3.5
    mul = st.uniform(cout, 1e-4, 3e-4).astype(np.float32)
    add = st.uniform(cout, -0.3, 0.3).astype(np.float32)
    for kind in (SUBM, STRIDED):
        _, nbr, _ = oracle.build_kmap(kind, coords, grid, nb)
        _check_conv(ctx, xq, wq, mul, add, kind == SUBM, nbr, nbr.shape[1] + 29)
    # a table with no structure
    n_out = 777
    rnd = (st.bits(27 * n_out) % np.uint64(len(coords))).astype(np.int32).reshape(27, n_out)
    rnd[st.uniform(27 * n_out, 0.0, 1.0).reshape(27, n_out) < 0.6] = -1
    _check_conv(ctx, xq, wq, mul, add, True, rnd, n_out)
    # nothing to do, and nothing but absent neighbours
    _check_conv(ctx, xq[:0], wq, mul, add, False, np.zeros((27, 0), np.int32), 8)
    v = _check_conv(ctx, xq, wq, mul, add, False, -np.ones((27, 70), np.int32), 70)
    assert np.array_equal(v, np.broadcast_to(add, v.shape))
    ctx.close()


def test_spconv_e4m3_exact_small_integers():
    """Operands that are small integers: every partial sum is an integer below 2^24, so fp32 accumulation is exact in
    any order and the GPU must match the oracle bit for bit -- a check of the format the matrix cores decode (a
    different exponent bias or special-value convention would scale or corrupt these)."""
    ctx = B.Context(16, 4096, 64 * 64 * 8, n_slots=1)
    cin, cout = 64, 64
    grid, nb = (10, 9, 5), 1
    coords = _rand_sites(77, grid, nb, 400)
    st = gen.Stream(5, 55)
    ints = np.array([0, 1, 2, 3, 4, 5, 6, 7, 8], np.float32)
    xv = ints[(st.bits(len(coords) * cin) % np.uint64(9)).astype(np.int64)].reshape(-1, cin) * np.where(st.uniform(len(coords) * cin).reshape(-1, cin) < 0.5, -1, 1)
    wv = ints[(st.bits(27 * cin * cout) % np.uint64(5)).astype(np.int64)].reshape(27, cin, cout) * np.where(st.uniform(27 * cin * cout).reshape(27, cin, cout) < 0.5, -1, 1)
    xq, wq = oracle.quantize_e4m3(xv.astype(np.float32), 1.0), oracle.quantize_e4m3(wv.astype(np.float32), 1.0)
    _, nbr, _ = oracle.build_kmap(SUBM, coords, grid, nb)
    one, zero = np.ones(cout, np.float32), np.zeros(cout, np.float32)
    exp = oracle.spconv_e4m3(xq, wq, one, zero, False, nbr)
    want = oracle.spconv(xv.astype(np.float32), wv.astype(np.float32), None, None, 0, nbr)     # the integers themselves
    assert np.array_equal(exp, want)
    n_out = nbr.shape[1]
    wp = torch.empty((27 * cin * cout,), dtype=torch.int8, device="cuda")
    ctx.pack_weights_i8(dev(wq.view(np.int8)), wp)
    out = torch.zeros((n_out, cout), dtype=torch.float32, device="cuda")
    ctx.spconv_e4m3(dev(xq), wp, cin, cout, dev(one), dev(zero), False, dev(nbr), torch.tensor([n_out], dtype=torch.int32, device="cuda"),
                    n_out, out)
    torch.cuda.synchronize()
    assert np.array_equal(out.cpu().numpy(), exp)
    ctx.close()


def test_spconv_e4m3_config2_level2_full_size():
    """The dominant layer of the front-view backbone (64 -> 64 submanifold at level 2) with quantised activations of
    the real chain, at full size."""
    cfg = get_config(2)
    br = cfg.branches[0]
    pts_np, _ = gen.make_frames(cfg)
    caps = default_capacities(br, len(pts_np))
    ctx = B.Context(len(pts_np), max(caps), cells_of(br.spec.grid, 1), n_slots=len(caps))
    runner = BranchRunner(ctx, br, cfg.dtype, len(pts_np), device_params(br.layers, gen.frame_seed(2, 0), cfg.dtype), capacities=caps)
    runner.run(dev(pts_np), None)
    ctx.status_sync()
    li = 5                                                              # first 64 -> 64 submanifold layer
    assert br.layers[li].cin == 64 and br.layers[li].cout == 64 and br.layers[li].kind == SUBM
    nbr, lv = runner.layer_map(li)
    n = int(lv.n.item())
    x16 = runner.acts[li - 1][:n].contiguous()
    xq = torch.empty((n, 64), dtype=torch.uint8, device="cuda")
    inv_s = 8.0
    ctx.quantize_e4m3(x16, inv_s, xq.view(-1))
    assert np.array_equal(xq.cpu().numpy(), oracle.quantize_e4m3(x16.float().cpu().numpy(), inv_s))
    wq = _rand_codes(4, (27, 64, 64), top=0x3F)
    st = gen.Stream(3, 3)
    mul = st.uniform(64, 1e-3, 2e-3).astype(np.float32)
    add = st.uniform(64, -0.1, 0.1).astype(np.float32)
    progress(f"spconv_e4m3 full size: {n} rows")
    _check_conv(ctx, xq.cpu().numpy(), wq, mul, add, True, nbr[:, :n].cpu().numpy(), lv.cap)
    ctx.close()
