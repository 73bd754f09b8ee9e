"""Which Poisson solve a shape takes, seen in the launches per phase: the passes
per axis transform y (and skip an axis of one node), the dense three-pass solve
has no phase of its own for y and always two for x.  Shapes from both sides of the
rule, thin sides, one fast side and many problems among them, and the two solves'
agreement: the same iterations within the FP32 tolerance of the parity tests
(1e-5 of the iterate's norm)."""
import numpy as np
import pytest

from oracle import grid as G
from synth import inputs
from test_gpu_parity import TOL, host, oracle, otdyn, rel, run_gpu, to_natural  # noqa: F401

pytestmark = pytest.mark.gpu

# X, Y, C, P, problems, dense three-pass solve
ROUTES = [
    (1, 180, 3, 16, 32, False),      # one axis, fast
    (1, 180, 1, 12, 32, False),
    (1, 60, 1, 12, 4, True),         # one axis, few nodes
    (32, 1, 3, 40, 16, True),        # many colours and times
    (32, 1, 1, 12, 256, False),
    (1, 64, 3, 40, 1, True),
    (1, 512, 1, 48, 1, False),       # a long fast y
    (150, 1, 3, 16, 1, True),        # times in registers, an odd length
    (1, 150, 1, 16, 1, True),
    (1, 300, 1, 8, 32, False),
    (1, 12, 3, 16, 64, False),
    (1, 64, 3, 16, 1, False),
    (180, 40, 3, 32, 4, False),      # one fast side
    (16, 100, 3, 32, 16, False),
    (24, 24, 3, 16, 64, False),      # many small ones
    (100, 64, 1, 10, 64, False),     # two fast sides, times without a register transform
    (200, 32, 1, 8, 64, False),      # a side of 32
    (32, 70, 1, 16, 64, False),
    (32, 20, 1, 8, 1, True),
    (16, 16, 3, 8, 1, True),
    (36, 36, 3, 16, 40, True),
    (50, 70, 3, 16, 1, True),
    (100, 64, 3, 12, 1, True),
    (2, 300, 3, 8, 4, True),         # thin x, long y
]


@pytest.mark.parametrize("route", ROUTES, ids=lambda r: "x".join(map(str, r[:5])))
def test_route_and_result(otdyn, route):  # noqa: F811
    X, Y, C, P, B, dense = route
    print(f"route {route}", flush=True)
    g = G.Grid(X, Y, C, P, (G.NEUMANN, G.NEUMANN, G.NEUMANN))
    pairs = [inputs.random_pair(3 + X + Y + P + (b % 2), X, Y, C) for b in range(B)]
    prob = run_gpu(otdyn, g, np.stack([p[0] for p in pairs]), np.stack([p[1] for p in pairs]), 3,
                   refine=1, batch=B)
    x = to_natural(g, *host(prob, B - 1))
    st = oracle(g, *pairs[B - 1], 3)
    for a in range(4):
        if st.x[a].size:
            assert rel(x[a], st.x[a]) < TOL, a
    otdyn.ot_dyn_profile(prob.plan, (1 << otdyn.OT_PHASE_COUNT) - 1)
    prob.step(1)
    phases = otdyn.ot_dyn_profile_read(prob.plan)
    solves = phases["tc"][1]
    assert solves in (1, 2)
    assert phases["xform_x"][1] == (2 * solves if dense or X > 1 else 0)
    assert phases["xform_y"][1] == (0 if dense or Y == 1 else 2 * solves)
    prob.close()
