"""Pressure and velocity on wide tiles (single 3D cases of 640 of them and
more, 4-byte fields) against the narrow tiles, which a serving batch always takes:
the same arithmetic term by term, so the fields are bitwise equal.  The grids
have remainders of 1 to 3 nodes of the 64 x 4 x 4 tiles on every axis, fewer
nodes than one tile in x and more than one, walls on every face, an open top,
and a block inside, at a face and across tiles; the smallest has just the 640
at which wide tiles start.  Reversed tiles cover the race check.  The
fields are rough on purpose (some cases diverge within the 5 steps, in the
reference too): they are compared from the initial state on."""
import numpy as np
import pytest

from paper_2512_01027_amd import binding as B
from paper_2512_01027_amd import workloads as W

pytestmark = pytest.mark.gpu

GRIDS = {
    "threshold": dict(n=(5, 160, 64)),
    "periodic": dict(n=(67, 75, 70)),
    "walls": dict(n=(130, 49, 69), wall=(1, 1, 1), gravity=(1e-6, 2e-6, -1e-5)),
    "walls_z": dict(n=(66, 54, 91), wall=(0, 0, 1), gravity=(0.0, 0.0, -1e-5)),
    "block": dict(n=(131, 45, 74), wall=(1, 1, 2), gravity=(0.0, 0.0, -1e-5), p_top=0.01,
                  block=((60, 9, 0), (69, 21, 6))),
    "block_inside": dict(n=(70, 81, 63), wall=(0, 1, 1), gravity=(0.0, -1e-5, 2e-6), block=((30, 20, 11), (40, 33, 29))),
}


@pytest.mark.parametrize("store,q", [("fp32", 27), ("fp16", 27), ("fp32", 19), ("bf16", 19)])
@pytest.mark.parametrize("name", sorted(GRIDS))
def test_wide_tiles_equal_narrow_bitwise(name, store, q):
    kw = dict(GRIDS[name])
    cfg = W.base_case(3, *kw.pop("n"), q_hydro=q, nu_heavy=0.05, nu_light=0.1, store=store, **kw)
    assert -(-cfg["nx"] // 64) * -(-cfg["ny"] // 4) * -(-cfg["nz"] // 4) >= 640
    phi, P, u = W.droplet(cfg, 0.3 * min(cfg["ny"], cfg["nz"]), center=(2.3, cfg["ny"] * 0.45, cfg["nz"] * 0.6))
    for a in range(3):
        u[a] += W.random_smooth(cfg, 7 + a, amp=0.01)
    P += W.random_smooth(cfg, 4, amp=1e-3)
    for order, steps in ((0, 0), (0, 1), (0, 2), (1, 5)):
        bt = B.Batch(1 << 30, store=store, max_slots=2)
        slot = bt.admit(cfg, phi, P, u, steps)
        bt.advance(max(steps, 1))
        assert bt.poll() == [slot]
        ref = bt.take(slot)
        bt.close()
        c = B.Case(cfg)
        c.set_tile_order(order)
        c.init_fields(phi, P, u)
        c.step(steps)
        out = c.read_fields()
        c.close()
        for nm, a, b in zip(("phi", "P", "u"), out, ref):
            assert np.array_equal(a, b, equal_nan=True), f"{name} {store} order {order} steps {steps}: {nm}"
