"""Convolutions whose XCDs take runs of rows in turn: every row of the level is computed, once, and none beyond it, at the edges of a
run, of a turn of eight runs and of the capacity."""
import pytest
import torch

from paper_2507_04123_amd import binding as B
from paper_2507_04123_amd.configs import EPI_NONE, F16

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cin,cout", [(64, 64), (64, 128), (128, 128), (16, 32), (32, 32), (32, 64), (64, 32)])
@pytest.mark.parametrize("n", [1, 511, 513, 1024, 8 * 512 - 1, 8 * 512 + 1, 8 * 1024 + 33, 16 * 1024, 32768 + 129, 66500])
def test_every_row_once(cin, cout, n):
    ctx = B.Context(16, 16, 64, n_slots=1)
    g = torch.Generator(device="cuda").manual_seed(n)
    for cap in (n, n + 700):
        x = torch.randn((cap, cin), generator=g, device="cuda").half()
        perm = torch.randperm(cap, generator=g, device="cuda").to(torch.int32)
        nbr = torch.full((27, cap), -1, dtype=torch.int32, device="cuda")
        nbr[13] = perm                                   # row i <- input row perm[i], by one tap of ones on a diagonal: exact
        w = torch.zeros((27, cin, cout), device="cuda")
        c = torch.arange(cout, device="cuda")
        w[13, c % cin, c] = 1.0
        wp = torch.empty_like(w, dtype=torch.float16)
        ctx.pack_weights(F16, w.half(), wp)
        y = torch.full((cap, cout), -7.0, dtype=torch.float16, device="cuda")
        ctx.spconv(F16, x, wp, None, None, EPI_NONE, nbr, torch.tensor([n], dtype=torch.int32, device="cuda"), cap, y,
                   w_layout=B.W_PACKED, map_hint=B.MAP_ANY)
        torch.cuda.synchronize()
        assert torch.equal(y[:n], x[perm[:n].long()][:, c % cin])
        assert (y[n:] == -7.0).all()
        ctx.status_sync()
