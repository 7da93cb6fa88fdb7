"""Which convolution calls of a list wait for one another, as the list's planning sees it (no GPU): the header it is written in,
compiled by itself, against the byte ranges in unbounded integers."""
import ctypes
import os
import subprocess

import pytest

from paper_2507_04123_amd import binding as B
from paper_2507_04123_amd import build as hip_build
from paper_2507_04123_amd.configs import F16, F32

_SHIM = """#include "conv_order.h"
extern "C" int ordered(const emc2_conv_call* a, const emc2_conv_call* b) { return emc2_ordered(emc2_touched_by(*a), emc2_touched_by(*b)); }
"""


@pytest.fixture(scope="module")
def ordered(tmp_path_factory):
    d = tmp_path_factory.mktemp("conv_order")
    (d / "shim.cpp").write_text(_SHIM)
    subprocess.run(["g++", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I", hip_build.CSRC, "-I", os.path.join(hip_build.ROOT, "include"),
                    str(d / "shim.cpp"), "-o", str(d / "shim.so")], check=True)
    f = ctypes.CDLL(str(d / "shim.so")).ordered
    return lambda a, b: bool(f(ctypes.byref(a), ctypes.byref(b)))


def _call(at, dt=F16, cap=100, n_in=100, cin=16, cout=16, **fields):
    """A call whose buffers lie a mebibyte apart from `at` on."""
    c = B.ConvCallC()
    names = ("d_out", "d_in", "d_w", "d_scale", "d_shift", "d_nbr", "d_n_out")
    for i, name in enumerate(names):
        setattr(c, name, at + (i << 20))
    c.capacity_out, c.n_in_rows, c.dtype, c.cin, c.cout = cap, n_in, dt, cin, cout
    for k, v in fields.items():
        setattr(c, k, v)
    return c


def _sizes(c):
    e = 4 if c.dtype == F32 else 2
    return {"d_out": c.capacity_out * c.cout * e, "d_in": min(c.n_in_rows, 2 ** 31 - 1) * c.cin * e, "d_w": 27 * c.cin * c.cout * e,
            "d_scale": 4 * c.cout, "d_shift": 4 * c.cout, "d_nbr": 27 * c.capacity_out * 4, "d_n_out": 4}


A, Z = 1 << 40, 1 << 41


@pytest.mark.parametrize("what", ["d_out", "d_in", "d_w", "d_scale", "d_shift", "d_nbr", "d_n_out"])
@pytest.mark.parametrize("dt", [F16, F32])
def test_whatever_another_call_writes(ordered, what, dt):
    """Each buffer of the second call at the first byte, the last one and beyond either end of the first call's output."""
    first = _call(A, dt=dt)
    n_out = _sizes(first)["d_out"]
    n = _sizes(_call(Z, dt=dt))[what]
    for to, waits in ((A, True), (A + n_out - 1, True), (A + n_out, False), (A - n + 1, True), (A - n, False)):
        second = _call(Z, dt=dt, **{what: to})
        assert ordered(first, second) == waits and ordered(second, first) == waits


def test_what_is_only_read_is_shared(ordered):
    first = _call(A)
    assert not ordered(first, _call(Z, d_in=first.d_in, d_w=first.d_w, d_scale=first.d_scale, d_nbr=first.d_nbr, d_n_out=first.d_n_out))


@pytest.mark.parametrize("rows", [1 << 31, 1 << 59, 1 << 60, 1 << 62, (1 << 63) - 1])
@pytest.mark.parametrize("cin", [4, 16, 64, 128])
def test_a_row_count_that_stands_for_no_limit(ordered, rows, cin):
    """Rows beyond 2^31 - 1 are refused by no check and clamped by the launch: the input still reaches as far as that."""
    first = _call(A)
    assert ordered(first, _call(Z, n_in=rows, cin=cin, d_in=A))
    assert ordered(first, _call(Z, n_in=rows, cin=cin, d_in=A - 4096))
    assert not ordered(first, _call(Z, n_in=rows, cin=cin, d_in=A + 1600 * 2))
    top = (1 << 64) - (1 << 24)              # a range that would pass the end of the address space ends there
    assert ordered(_call(top), _call(Z, n_in=rows, cin=cin, d_in=top))


@pytest.mark.parametrize("cap", [1 << 57, 1 << 60, (1 << 63) - 1])
def test_a_capacity_whose_bytes_do_not_fit_64_bits(ordered, cap):
    assert ordered(_call(A, cap=cap, cout=64), _call(Z, d_in=A))
    assert ordered(_call(A, cap=cap, cout=64), _call(Z, d_in=A + (1 << 30)))
