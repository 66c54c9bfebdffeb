"""The BF16 encoder against rounding to nearest-even on the host, through the
moment kernel: a node's populations along x are set, by a restart image, to the
BF16 pieces of a binary32 value, whose sum (the xx moment) is that value
exactly; the kernel stores it in BF16 in the case's device memory.  Ties to
even and odd, one unit to either side of a tie, carries into the exponent, the
smallest normal numbers, the largest (to infinity from the tie on), zero,
infinity and NaN, in both signs, and random values."""
import ctypes as C

import numpy as np
import pytest

from paper_2512_01027_amd import binding as B
from paper_2512_01027_amd import workloads as W

pytestmark = pytest.mark.gpu

NX, NY = 64, 40


def _rne(bits):
    """Upper 16 bits of binary32 patterns, rounded to nearest-even (no NaNs)."""
    b = bits.astype(np.uint64)
    return ((b + 0x7FFF + ((b >> 16) & 1)) >> 16).astype(np.uint16)


def _values():
    rng = np.random.default_rng(11)
    up = np.array([0x3F80, 0x3F81, 0x3FFF, 0x0900, 0x0980, 0x09FF, 0x7F7E, 0x7F7F, 0x4049, 0x7F00], np.uint32) << 16
    low = np.array([0, 1, 0x7FFF, 0x8000, 0x8001, 0xFFFF], np.uint32)
    edge = (up[:, None] | low[None, :]).ravel()
    rand = rng.integers(0x10000000, 0x7F000000, NX * NY // 2 - edge.size - 8, dtype=np.uint32)
    v = np.concatenate([edge, rand])
    return np.concatenate([v, v | np.uint32(0x80000000)]).view(np.float32)


def _pieces(v):
    """v = a + b + c exactly, each a BF16 number (8 of its 24 bits)."""
    cut = lambda x: (x.view(np.uint32) & np.uint32(0xFFFF0000)).view(np.float32)  # noqa: E731
    a = cut(v)
    b = cut((v - a).astype(np.float32))
    c = ((v - a) - b).astype(np.float32)
    assert (cut(c) == c).all() and ((a + b) + c == v).all()
    return a, b, c


def test_moment_kernel_rounds_to_nearest_even():
    v = _values()
    special = np.array([0.0, np.inf, -np.inf, np.nan], np.float32)
    cfg = W.base_case(2, NX, NY, store="bf16")
    case = B.Case(cfg)
    z = np.zeros(NX * NY)
    case.init_fields(z, z, np.zeros(2 * NX * NY))
    N = NX * NY  # rows of 64 nodes need no padding
    blob = bytearray(case.checkpoint())
    head = 8 + 8 + C.sizeof(B.Params) + 8 + 3 * 8
    pops = np.frombuffer(blob, dtype=np.uint16, offset=head, count=18 * N).reshape(18, N)
    pops[:] = 0
    g = pops[9:]
    a, b, c = _pieces(v)
    for d, x in zip((1, 2, 5), (a, b, c)):  # +x, -x and a diagonal, in the order they are summed
        g[d, :v.size] = (x.view(np.uint32) >> 16).astype(np.uint16)
    g[1, v.size:v.size + 4] = (special.view(np.uint32) >> 16).astype(np.uint16)
    aux = np.frombuffer(blob, dtype=np.float32, offset=head + 18 * N * 2)
    aux[:] = 0  # the references of the codec
    case.restore(bytes(blob))
    case.read_fields()
    # M2 follows h, g, two of P, two of phi, u* and P* (each section on 256 bytes)
    up = lambda n: -(-n // 256) * 256  # noqa: E731
    off = 2 * up(9 * N * 2) + 4 * up(N * 4) + up(2 * N * 4) + up(N * 4)
    base = (-case._arena.data_ptr()) % 256
    m2 = case._arena[base + off: base + off + 4 * N].cpu().numpy().view(np.uint32)
    xx = (m2 & 0xFFFF).astype(np.uint16)  # the low half of the first word
    want = _rne(v.view(np.uint32))
    bad = np.flatnonzero(xx[:v.size] != want)
    assert bad.size == 0, [(hex(v.view(np.uint32)[i]), hex(xx[i]), hex(want[i])) for i in bad[:8]]
    zero, pinf, ninf, nan = xx[v.size:v.size + 4]
    assert zero == 0 and pinf == 0x7F80 and ninf == 0xFF80
    assert nan & 0x7F80 == 0x7F80 and nan & 0x40
    case.close()
