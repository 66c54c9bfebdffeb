"""2D steps whose collide kernel rebuilds P and u from a 3-node halo of P* and
u*: grids whose last tile (64 x 4 nodes) holds 1 to 3 nodes or ends 1 to 3
nodes short, down to the smallest fused ones (3 x 3), periodic, with walls and
with an open top, both collisions, against the FP64 CPU reference (1e-10, the
parity tests' bound)."""
import numpy as np
import pytest

import oracle
from paper_2512_01027_amd import binding as B
from paper_2512_01027_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("collision", ["filter", "bgk"])
@pytest.mark.parametrize("wall", [(0, 0, 0), (1, 0, 0), (0, 1, 0), (1, 1, 0), (0, 2, 0), (1, 2, 0)])
@pytest.mark.parametrize("n", [(3, 3), (4, 5), (61, 7), (62, 6), (63, 5), (64, 4), (65, 9), (66, 3), (67, 10), (130, 8)])
def test_fused_2d_matches_oracle(n, wall, collision):
    cfg = W.base_case(2, *n, wall=wall, gravity=(1e-6, -1e-5, 0.0), nu_heavy=0.1, nu_light=0.15, sigma=0.01,
                      rho_heavy=50.0, p_top=0.02 if wall[1] == 2 else 0.0, collision=collision, store="fp64")
    phi, P, u = W.droplet(cfg, 0.3 * n[1] + 0.4, center=(n[0] * 0.47, n[1] * 0.53, 0.0))
    phi = np.clip(phi + W.random_smooth(cfg, 5, amp=0.02), 0, 1)
    for a in range(2):
        u[a] += W.random_smooth(cfg, 6 + a, amp=0.01)
    P += W.random_smooth(cfg, 14, amp=1e-3) + cfg["p_top"]
    g = B.Case(cfg)
    g.init_fields(phi, P, u)
    o = oracle.OracleCase(cfg)
    o.init_fields(phi, P, u)
    for steps in (1, 2, 5):
        g.step(steps - g.steps_done)
        o.step(steps - o.diagnostics()["step"])
        for nm, a, b in zip(("phi", "P", "u"), g.read_fields(), o.read_fields()):
            err = np.abs(a - b).max() / max(np.abs(b).max(), 1e-12)
            assert err < 1e-10, (n, wall, steps, nm, err)
