"""Dense three-pass Poisson solve (csrc/dense3.hip) at the edges of its tiles and
launch rules, against the FP64 CPU oracle at the tolerance of the other parity
tests (1e-5 of the iterate's norm, FP32 iterations of the same recurrence)."""
import numpy as np
import pytest

from oracle import grid as G
from synth import inputs
from test_gpu_parity import TOL, host, oracle, otdyn, rel, run_gpu, to_natural  # noqa: F401

pytestmark = pytest.mark.gpu

N, PER = G.NEUMANN, G.PERIODIC
SHAPES = [
    # X, Y, C, P, bc, problems
    (17, 1, 1, 5, (N, N, N), 2),           # one row, folded x just past a tile
    (1, 17, 1, 6, (N, N, N), 1),           # one column
    (16, 15, 3, 7, (N, N, PER), 1),        # unfolded, full and partial tile
    (15, 33, 4, 9, (PER, N, PER), 2),      # C = 4, folded odd y over two tiles
    (34, 20, 2, 13, (N, PER, N), 1),       # several time groups, periodic y
    (65, 18, 3, 17, (N, N, PER), 1),       # P over one time tile
    (19, 21, 1, 40, (N, N, N), 1),         # P past the matrices held in registers
    (21, 19, 1, 64, (PER, N, N), 1),       # the most times
    (21, 19, 1, 65, (N, N, N), 1),         # one more: the general passes
    (300, 11, 1, 5, (N, N, N), 1),         # two output tiles per wave, x
    (11, 300, 3, 20, (N, PER, PER), 1),    # two output tiles per wave, y, P over a tile
    (530, 7, 1, 4, (N, N, N), 1),          # past the longest side: the general passes
    (512, 3, 2, 12, (PER, N, PER), 1),     # the longest side, unfolded
    (20, 18, 5, 6, (N, N, PER), 1),        # C = 5: the general passes
    (26, 22, 3, 12, (N, N, PER), 24),      # all colours per block of the y and time pass
]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s[:4])))
def test_dense_solve_matches_oracle(otdyn, shape):  # noqa: F811
    X, Y, C, P, bc, B = shape
    print(f"dense solve {shape}", flush=True)
    g = G.Grid(X, Y, C, P, bc)
    pairs = [inputs.random_pair(11 + X + Y + P + b, X, Y, C) for b in range(B)]
    prob = run_gpu(otdyn, g, np.stack([p[0] for p in pairs]), np.stack([p[1] for p in pairs]), 6,
                   refine=1, batch=B)
    for b in sorted({0, B - 1}):
        x = to_natural(g, *host(prob, b))
        st = oracle(g, *pairs[b], 6)
        for a in range(4):
            if st.x[a].size:
                assert rel(x[a], st.x[a]) < TOL, (b, a)
    prob.close()
