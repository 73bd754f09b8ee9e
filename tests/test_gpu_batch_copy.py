"""The packed states of a batch whose members' pieces start at every alignment:
a state put in and taken out again is the same, and each group's single plan gets
the same boundary densities."""
import numpy as np
import pytest

from test_gpu_parity import otdyn  # noqa: F401

pytestmark = pytest.mark.gpu

DIMS = [(7, 5, 3, 4), (64, 1, 1, 16), (9, 1, 1, 5), (7, 5, 3, 4), (64, 1, 1, 16), (5, 1, 1, 3), (9, 1, 1, 5)]


def test_packed_state_round_trip(otdyn):  # noqa: F811
    import torch
    print("batch copy", flush=True)
    o = otdyn
    base = o.ot_dyn_default_desc(1, 1, 1, 2)
    base.bc[0], base.bc[1], base.bc[2] = 1, 1, 1          # no walls along an axis of several nodes
    bt = o.Batch(base, DIMS, "cuda")
    rng = np.random.default_rng(3)
    h = [[rng.random(X * Y * C).astype(np.float32) + 0.1 for X, Y, C, P in DIMS] for _ in range(2)]
    h = [[v / v.mean() for v in q] for q in h]
    bt.set_boundary(*h)
    F = [np.concatenate([h[0][i], rng.random((P - 1) * X * Y * C), h[1][i]]).astype(np.float32)
         for i, (X, Y, C, P) in enumerate(DIMS)]
    M = [rng.standard_normal((3, P * X * Y * C)).astype(np.float32) for X, Y, C, P in DIMS]
    for i, (X, Y, C, P) in enumerate(DIMS):
        if C == 1:
            M[i][2] = 0                                   # no colour faces
    want = [m.copy() for m in M]
    for i, (X, Y, C, P) in enumerate(DIMS):
        if Y == 1:
            want[i][1] = 0                                # one node along y: its faces are walls
    F, M, want = np.concatenate(F), *(np.concatenate([m.reshape(-1) for m in q]) for q in (M, want))
    bt.set_state(torch.as_tensor(F).cuda(), torch.as_tensor(M).cuda(), o.OT_INIT_PRIMAL)
    F2, M2 = bt.packed_state()
    assert np.array_equal(F2.cpu().numpy(), F)
    assert np.array_equal(M2.cpu().numpy(), want)
    bt.close()
