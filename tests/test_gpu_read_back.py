"""pulbm_read_fields moves the fields in pieces of 1 MiB, two to each of up to 8
threads: bit for bit the allocation-free read-back, which copies whole fields,
at sizes of one short piece, of two pieces, and of two, four and eight threads
with a ragged last piece and padded rows; any of the arrays left out; and
several threads that read their own cases at once."""
import ctypes as C
import threading

import numpy as np
import pytest
import torch

from paper_2512_01027_amd import binding as B
from paper_2512_01027_amd import workloads as W

pytestmark = pytest.mark.gpu


def _case(n, store, seed=3, **kw):
    cfg = W.base_case(2 if n[2] == 1 else 3, *n[: 2 if n[2] == 1 else 3], sigma=0.01, store=store)
    rng = np.random.default_rng(seed)
    N = n[0] * n[1] * n[2]
    shape = W.droplet(cfg, 5.0)[0].shape
    dim = cfg["dim"]
    c = B.Case(cfg, **kw)
    c.init_fields(rng.uniform(0, 1, N).reshape(shape), rng.uniform(-1e-3, 1e-3, N).reshape(shape),
                  rng.uniform(-1e-2, 1e-2, dim * N).reshape((dim,) + shape))
    return c


def _same(a, b):
    return all(np.array_equal(x, y, equal_nan=True) for x, y in zip(a, b))


@pytest.mark.parametrize("store", ["fp64", "fp32", "fp16"])
@pytest.mark.parametrize("n", [(5, 3, 1), (37, 29, 1), (257, 255, 1), (260, 253, 1), (61, 47, 33), (131, 83, 51), (1101, 967, 1), (191, 93, 92)])
def test_read_fields_equals_noalloc(n, store):
    c = _case(n, store)
    for steps in (0, 3):
        c.step(steps)
        want = c.read_fields_noalloc()
        assert _same(c.read_fields(), want)
    phi, P, u = (np.full(a.size, 7.0) for a in want)
    dp = lambda a: a.ctypes.data_as(C.POINTER(C.c_double))  # noqa: E731
    assert c.lib.pulbm_read_fields(c._h, None, dp(P), None) == B.OK
    assert c.lib.pulbm_read_fields(c._h, dp(phi), None, dp(u)) == B.OK
    assert c.lib.pulbm_read_fields(c._h, None, None, None) == B.OK
    assert _same((phi, P, u), (a.reshape(-1) for a in want))
    c.close()


def test_read_fields_from_several_threads():
    cs = [_case(n, "fp32", seed=i) for i, n in enumerate([(131, 83, 51), (61, 47, 33), (1101, 967, 1), (37, 29, 1)] * 2)]
    want = [c.read_fields_noalloc() for c in cs]
    bad = []

    def loop(i):
        torch.cuda.set_device(0)
        for _ in range(5):
            if not _same(cs[i].read_fields(), want[i]):
                bad.append(i)

    ts = [threading.Thread(target=loop, args=(i,)) for i in range(len(cs))]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    for c in cs:
        c.close()
    assert not bad
