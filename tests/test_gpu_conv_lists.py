"""emc2_spconv_list against the same calls one by one, bit for bit: calls that share a launch, calls that wait for one another through
any of their buffers, more than a launch holds, a refused one in between."""
import pytest
import torch

from paper_2507_04123_amd import binding as B
from paper_2507_04123_amd.configs import BF16, EPI_AFFINE, EPI_AFFINE_RELU, F16, F32
from test_gpu_stacks import _kernels_in

pytestmark = pytest.mark.gpu


class _Pool:
    def __init__(self, seed):
        self.g = torch.Generator(device="cuda").manual_seed(seed)
        self.ctx, self.keep = [B.Context(16, 16, 64, n_slots=1) for _ in range(2)], []
        self.maps, self.outs = [], []     # places of the calls' maps in `keep`; the calls' outputs

    def rows(self, n, ch, dt):
        td = {F16: torch.float16, BF16: torch.bfloat16, F32: torch.float32}[dt]
        self.keep.append(torch.randn((n, ch), generator=self.g, device="cuda").to(td))
        return self.keep[-1]

    def call(self, x, y, cin, cout, dt, n=None, hint=B.MAP_ANY, ctx=0):
        """x -> y (rows of their buffers), a random third of the entries of the map there."""
        cap = y.shape[0]
        n = cap if n is None else n
        nbr = torch.randint(-2 * x.shape[0], x.shape[0], (27, cap), generator=self.g, device="cuda", dtype=torch.int32)
        w = (torch.randn((27, cin, cout), generator=self.g, device="cuda") * 0.1).to(x.dtype)
        mfma = dt != F32 and self.ctx[0].lib.emc2_spconv_uses_mfma(dt, cin, cout)
        if mfma:
            wp = torch.empty_like(w)
            self.ctx[0].pack_weights(dt, w, wp)
            w = wp
        sc, sh = torch.rand(cout, generator=self.g, device="cuda"), torch.randn(cout, generator=self.g, device="cuda")
        nn = torch.tensor([n], dtype=torch.int32, device="cuda")
        self.maps.append(len(self.keep))
        self.outs.append(y)
        self.keep += [nbr, w, sc, sh, nn]
        c = B.ConvCallC()
        c.ctx, c.d_in, c.d_w, c.d_scale, c.d_shift = self.ctx[ctx].h, x.data_ptr(), w.data_ptr(), sc.data_ptr(), sh.data_ptr()
        c.d_nbr, c.d_n_out, c.d_out, c.capacity_out, c.n_in_rows = nbr.data_ptr(), nn.data_ptr(), y.data_ptr(), cap, x.shape[0]
        c.dtype, c.w_layout, c.epilogue, c.map_hint, c.cin, c.cout = dt, (B.W_PACKED if mfma else B.W_PLAIN), EPI_AFFINE_RELU, hint, cin, cout
        return c


def _both(pool, calls, outs):
    """Outputs of the calls one by one, then as a list, from the same buffers."""
    start = [y.clone() for y in outs]
    for c in calls:
        B.spconv_list((B.ConvCallC * 1)(c), 1)
    torch.cuda.synchronize()
    exp = [y.clone() for y in outs]
    for y, s in zip(outs, start):
        y.copy_(s)
    arr = (B.ConvCallC * len(calls))(*calls)
    B.spconv_list(arr, len(calls))
    torch.cuda.synchronize()
    for i, (y, e) in enumerate(zip(outs, exp)):
        assert torch.equal(y, e), i
    for c in pool.ctx:
        c.status_sync()
    return arr


@pytest.mark.parametrize("dt", [F16, BF16])
@pytest.mark.parametrize("branches", [2, 3, 4, 5])
def test_branches_share_launches(dt, branches):
    p = _Pool(branches)
    calls, outs = [], []
    for b in range(branches):       # 4 -> 16 -> 32 -> 32 -> 64 -> 32 each, of other sizes; one of them without a row
        n = (700, 1, 5000, 33, 260)[b]
        x = p.rows(n, 4, dt)
        for cin, cout in ((4, 16), (16, 32), (32, 32), (32, 64), (64, 32)):
            y = p.rows(n + 3 * cin, cout, dt)
            calls.append(p.call(x, y, cin, cout, dt, n=0 if n == 33 else None, ctx=b % 2))
            outs.append(y)
            x = y
    arr = _both(p, calls, outs)
    assert _kernels_in(lambda: B.spconv_list(arr, len(calls))) == 5 * ((branches + 3) // 4)


def test_what_waits_stays_in_order():
    p = _Pool(9)
    a, b, c, d = (p.rows(900, 16, F16) for _ in range(4))
    # b from a, c from a, a from c (read by both before), c again, d from the new a, then a call whose rows overlap c's tail
    tail = c[800:]
    calls = [p.call(a, b, 16, 16, F16), p.call(a, c, 16, 16, F16), p.call(c, a, 16, 16, F16), p.call(b, c, 16, 16, F16),
             p.call(a, d, 16, 16, F16), p.call(d, tail, 16, 16, F16), p.call(b, p.rows(900, 16, F16), 16, 16, F16)]
    _both(p, calls, [a, b, c, d])


# (fp32 calls never share a launch; 16-bit ones of one shape do, by one of three kernels)
@pytest.mark.parametrize("cin,cout", [(4, 16), (16, 16), (16, 32), (32, 32), (32, 64), (64, 32)])
@pytest.mark.parametrize("what", ["d_in", "no limit", "d_w", "d_scale", "d_shift", "d_nbr", "d_n_out", "d_out", None])
def test_buffers_that_an_earlier_call_of_the_list_writes(cin, cout, what):
    """Two calls of one kernel, the second of which reads the first one's output as `what`, wait for each other: two launches, where
    calls that share nothing take one.  The values the second finds there before the first is done are valid and give other results."""
    p = _Pool(cin + cout)
    x, z = p.rows(300, cin, F16), p.rows(40, cout, F16)
    y = p.rows(4096, cout, F16)                # room for a map of 40 rows and for every shape's weights
    first, second = p.call(x, y, cin, cout, F16), p.call(x, z, cin, cout, F16)
    if what == "d_nbr":                        # a map before; afterwards -1.0 everywhere, whose bits are a negative entry: no neighbour
        sc, sh = torch.zeros(cout, device="cuda"), torch.full((cout,), -1.0, device="cuda")
        p.keep += [sc, sh]
        first.d_scale, first.d_shift, first.epilogue = sc.data_ptr(), sh.data_ptr(), EPI_AFFINE
        y.view(torch.int32).view(-1)[: 27 * 40] = p.keep[p.maps[1]].view(-1)
    if what == "d_n_out":                      # five rows before; afterwards a number beyond the capacity: all of them
        sc, sh = torch.zeros(cout, device="cuda"), torch.ones(cout, device="cuda")
        p.keep += [sc, sh]
        first.d_scale, first.d_shift = sc.data_ptr(), sh.data_ptr()
        y.view(torch.int32)[0, 0] = 5
    if what == "no limit":
        second.d_in, second.n_in_rows = y.data_ptr(), 1 << 62
    elif what == "d_out":                      # its rows are some of the first one's
        second.d_out = y[1000:].data_ptr()
    elif what is not None:
        setattr(second, what, y.data_ptr())
    arr = (B.ConvCallC * 2)(first, second)
    assert _kernels_in(lambda: B.spconv_list(arr, 2)) == (1 if what is None else 2)
    _both(p, [first, second], [y, z])


def test_list_of_more_calls_than_are_planned():
    """Over 64 calls: one by one, in the order of the list."""
    p = _Pool(66)
    bufs = [p.rows(200 + i, 16, F16) for i in range(4)]
    calls = [p.call(bufs[i % 4], bufs[(i + 1) % 4], 16, 16, F16, ctx=i % 2) for i in range(33)]
    calls += [p.call(bufs[i % 3], p.rows(100, 16, F16), 16, 16, F16) for i in range(33)]
    arr = _both(p, calls, bufs + p.outs[-33:])
    assert _kernels_in(lambda: B.spconv_list(arr, len(calls))) == 66
    assert _kernels_in(lambda: B.spconv_list((B.ConvCallC * 33)(*calls[33:]), 33)) == 9


def test_refused_call_in_a_list():
    """Calls in front of it are issued, it and those behind it are not, those of its kernel among them."""
    p = _Pool(5)
    x = p.rows(500, 4, F16)
    ys = [p.rows(500, 16, F16) for _ in range(3)]
    calls = [p.call(x, y, 4, 16, F16) for y in ys]
    start = [y.clone() for y in ys]
    calls[1].cin = 0
    with pytest.raises(B.Emc2Error, match="channels outside"):
        B.spconv_list((B.ConvCallC * 3)(*calls), 3)
    torch.cuda.synchronize()
    assert not torch.equal(ys[0], start[0]) and torch.equal(ys[1], start[1]) and torch.equal(ys[2], start[2])
