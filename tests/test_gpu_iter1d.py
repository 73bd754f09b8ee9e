"""Whole iterations of one-axis problems in one launch against the same
iterations step by step (a plan whose phases are timed takes those), over every
length and number of steps that has them, both x boundary conditions, duals with
all components, iterations on both sides of the refinement and of a launch's
limit, and a batch group with frozen members.

Both evaluate the same FP32 expressions per node; the FP64 spatial-DC line is
summed in another order, which can move its FP32 rounding by an ulp (6e-8 of
it) an iteration, and the iteration does not expand differences: n iterations
stay within 1e-7 n of the iterates' norm."""
import numpy as np
import pytest

from synth import inputs
from test_gpu_parity import otdyn, rel  # noqa: F401

pytestmark = pytest.mark.gpu


def _run(o, X, P, per, iters, timed, dual, carry, batch):
    import torch
    d = o.ot_dyn_default_desc(X, 1, 1, P)
    d.bc[0] = 1 if per else 0
    d.tau, d.sigma, d.batch, d.carry_refine = 3.0, 0.33, batch, carry
    p = o.Problem(d, "cuda")
    pairs = [inputs.random_pair(X + P + b, X, 1, 1) for b in range(batch)]
    for q in range(2):
        assert pairs[0][q].shape == (1, 1, X)
    p.set_boundary(*(torch.as_tensor(np.stack([a[q] for a in pairs]).astype(np.float32)) for q in range(2)))
    p.init(o.OT_INIT_COLD)
    if dual:
        rng = np.random.default_rng(5)
        b = torch.as_tensor(0.01 * rng.standard_normal(p.get_dual().shape).astype(np.float32)).cuda()
        p.set_dual(b)
    if timed:
        o.ot_dyn_profile(p.plan, 1)
    p.step(iters)
    out = [t.double().cpu().numpy() for t in (*p.state(), p.get_dual(), p.get_dual_bar())]
    p.close()
    return out


@pytest.mark.parametrize("per", [False, True], ids=["neumann", "periodic"])
@pytest.mark.parametrize("P", [8, 16, 32])
@pytest.mark.parametrize("X", [64, 100, 128, 180, 256, 360])
@pytest.mark.parametrize("iters,dual,carry,batch", [(7, True, 3, 3), (131, False, 2, 1)])
def test_whole_iterations_equal_step_by_step(otdyn, X, P, per, iters, dual, carry, batch):  # noqa: F811
    print(f"whole iterations {X}x{P} per={per} {iters}", flush=True)
    a = _run(otdyn, X, P, per, iters, False, dual, carry, batch)
    b = _run(otdyn, X, P, per, iters, True, dual, carry, batch)
    for x, y in zip(a, b):
        if np.any(y):
            assert rel(x, y) < 1e-7 * iters
        else:
            assert not np.any(x)
