"""Pressure and velocity on wide tiles against the narrow tiles, in the
read-back itself: a large grid made of three copies of a small one along a
periodic axis takes wide tiles (640 of them and more) where the small one takes
narrow ones, and holds the small one's fields three times, bit for bit, at the
initial state and after steps.  Remainders of 2 and 3 nodes of the 64 x 4 x 4
tiles, periodic, walls and an open top."""
import numpy as np
import pytest

from paper_2512_01027_amd import binding as B
from paper_2512_01027_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("store,q", [("fp32", 27), ("fp16", 27), ("fp32", 19), ("bf16", 19)])
@pytest.mark.parametrize("wall", [(0, 0, 0), (1, 0, 1), (0, 0, 2)])
def test_copies_of_a_narrow_grid(wall, store, q):
    nx, ny, nz = 130, 42, 47
    tiles = lambda y: -(-nx // 64) * -(-y // 4) * -(-nz // 4)  # noqa: E731
    assert tiles(ny) < 640 <= tiles(3 * ny)
    kw = dict(q_hydro=q, wall=wall, gravity=(1e-6, 2e-6, -1e-5), p_top=0.01 if wall[2] == 2 else 0.0, nu_heavy=0.1,
              nu_light=0.15, sigma=0.005, rho_heavy=50.0, store=store)
    small, large = W.base_case(3, nx, ny, nz, **kw), W.base_case(3, nx, 3 * ny, nz, **kw)
    phi, P, u = W.droplet(small, 12.0, center=(63.0, 20.0, 24.0))
    for a in range(3):
        u[a] += W.random_smooth(small, 7 + a, amp=0.01)
    P += W.random_smooth(small, 4, amp=1e-3) + small["p_top"]
    three = lambda f: np.concatenate([f] * 3, axis=-2)  # noqa: E731
    s, c = B.Case(small), B.Case(large)
    s.init_fields(phi, P, u)
    c.init_fields(three(phi), three(P), three(u))
    for steps in (0, 1, 2, 5):
        s.step(steps - s.steps_done)
        c.step(steps - c.steps_done)
        for nm, x, y in zip(("phi", "P", "u"), c.read_fields(), s.read_fields()):
            assert np.isfinite(y).all()
            assert np.array_equal(x, three(y)), (steps, nm)
    s.close()
    c.close()
