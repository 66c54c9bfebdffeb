"""2D cases whose collide kernel rebuilds P and u, in every storage width.

- What the collide stores for the next step (P, and in 2-byte storage u, the
  codec's reference) is bit for bit what the separate pressure and velocity
  kernels form: those run in a read-back, so a case read at step k is held
  against the restart image, at step k + 1, of one that was never read.  Grids
  whose last tile (64 x 4 nodes) holds 1 to 3 nodes or ends 1 to 3 nodes short,
  periodic, with walls and with an open top, both collisions.
- In a serving batch that mixes them with cases that keep the separate kernels
  (a solid block inside), joining and leaving so that the table holds either
  kind alone and both, every case is bit for bit what it is alone.
"""
import ctypes as C

import numpy as np
import pytest

from paper_2512_01027_amd import binding as B
from paper_2512_01027_amd import workloads as W

pytestmark = pytest.mark.gpu

STORES = ["fp64", "fp32", "fp16", "bf16"]


def _setup(n, store, wall=(0, 0, 0), collision="filter", block=None, seed=5):
    cfg = W.base_case(2, *n, wall=wall, gravity=(1e-6, -1e-5, 0.0), nu_heavy=0.1, nu_light=0.15, sigma=0.01,
                      rho_heavy=50.0, p_top=0.02 if wall[1] == 2 else 0.0, collision=collision, store=store, block=block)
    phi, P, u = W.droplet(cfg, 0.3 * n[1] + 0.4, center=(n[0] * 0.47, n[1] * 0.53, 0.0))
    phi = np.clip(phi + W.random_smooth(cfg, seed, amp=0.02), 0, 1)
    for a in range(2):
        u[a] += W.random_smooth(cfg, seed + 1 + a, amp=0.01)
    P += W.random_smooth(cfg, seed + 9, amp=1e-3) + cfg["p_top"]
    return cfg, (phi, P, u)


def _image_fields(c, store):
    """P and (2-byte storage) u of a restart image: a header, the populations,
    P, the phi and the u of the step before, in rows padded to 32 nodes."""
    blob = c.checkpoint()
    nx, ny = c.params.nx, c.params.ny
    N = -(-nx // 32) * 32 * ny
    sb, at = {"fp64": (8, np.float64), "fp32": (4, np.float32), "fp16": (2, np.float32), "bf16": (2, np.float32)}[store]
    head = 8 + 8 + C.sizeof(B.Params) + 8 + 3 * 8
    aux = np.frombuffer(blob, dtype=at, offset=head + 18 * N * sb)
    assert aux.size == 4 * N
    rows = aux.reshape(4, ny, -1)[:, :, :nx]
    return rows[0], rows[2:]  # (u is not kept up in 4- and 8-byte storage)


@pytest.mark.parametrize("store", STORES)
@pytest.mark.parametrize("collision", ["filter", "bgk"])
@pytest.mark.parametrize("wall", [(0, 0, 0), (1, 1, 0), (0, 2, 0)])
@pytest.mark.parametrize("n", [(3, 3), (61, 7), (63, 5), (65, 9), (67, 10), (130, 8)])
def test_collide_stores_what_the_separate_kernels_form(n, wall, collision, store):
    cfg, f = _setup(n, store, wall, collision)
    a, b = B.Case(cfg), B.Case(cfg)
    a.init_fields(*f)
    b.init_fields(*f)
    for k in range(4):
        _, P, u = a.read_fields()
        b.step(1)
        Pi, ui = _image_fields(b, store)
        assert np.array_equal(Pi, P[0], equal_nan=True), (k, "P")
        if store in ("fp16", "bf16"):
            assert np.array_equal(ui, u[:, 0], equal_nan=True), (k, "u")
        a.step(1)
    a.close()
    b.close()


@pytest.mark.parametrize("store", STORES)
def test_batch_of_both_kinds(store):
    kinds = [_setup((64, 40), store, (1, 1, 0)), _setup((70, 33), store, (1, 1, 0), block=((20, 0, 0), (26, 9, 1))),
             _setup((37, 29), store, seed=8), _setup((45, 31), store, (0, 2, 0), block=((8, 4, 0), (11, 9, 1)))]
    # (case, steps, admitted after): only the first kind, both, only the second, both
    plan = [(0, 29, 0), (1, 43, 8), (3, 61, 24), (2, 24, 56)]
    want = []
    for k, steps, _ in plan:
        c = B.Case(kinds[k][0])
        c.init_fields(*kinds[k][1])
        c.step(steps)
        want.append(c.read_fields())
        c.close()
    bt = B.Batch(1 << 28, store=store, max_slots=4)
    slots, got, t = {}, {}, 0
    while len(got) < len(plan):
        for i, (k, steps, after) in enumerate(plan):
            if after == t:
                slots[bt.admit(kinds[k][0], *kinds[k][1], steps)] = i
        bt.advance(8)
        t += 8
        for s in bt.poll():
            got[slots.pop(s)] = bt.take(s)
    bt.close()
    for i, w in enumerate(want):
        for nm, x, y in zip(("phi", "P", "u"), got[i], w):
            assert np.array_equal(x, y, equal_nan=True), (i, nm)
