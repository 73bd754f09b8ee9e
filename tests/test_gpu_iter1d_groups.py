"""Whole iterations of one-axis problems (one launch for a run of iterations) and
the same iterations step by step share every expression and every order of a sum,
so their states, duals and extrapolated duals are equal bit for bit: over all
lengths with whole iterations, with more problems than the long ones are iterated
one by one for, and in a batch group whose members certify at different checks and
are frozen while the others go on."""
import numpy as np
import pytest

from synth import inputs
from test_gpu_batch import hue_problems, periodic_desc
from test_gpu_parity import otdyn  # noqa: F401

pytestmark = pytest.mark.gpu


def _run(o, X, P, per, iters, timed, batch):
    import torch
    d = o.ot_dyn_default_desc(X, 1, 1, P)
    d.bc[0] = 1 if per else 0
    d.tau, d.sigma, d.batch, d.carry_refine = 3.0, 0.33, batch, 4
    p = o.Problem(d, "cuda")
    pairs = [inputs.random_pair(X + P + b, X, 1, 1) for b in range(batch)]
    p.set_boundary(*(torch.as_tensor(np.stack([a[q] for a in pairs]).astype(np.float32)) for q in range(2)))
    p.init(o.OT_INIT_COLD)
    rng = np.random.default_rng(5)
    p.set_dual(torch.as_tensor(0.01 * rng.standard_normal(p.get_dual().shape).astype(np.float32)).cuda())
    if timed:                                  # a plan whose phases are timed goes step by step
        o.ot_dyn_profile(p.plan, 1)
    p.step(iters)
    out = [t.cpu().numpy() for t in (*p.state(), p.get_dual(), p.get_dual_bar())]
    p.close()
    return out


@pytest.mark.parametrize("per", [False, True], ids=["neumann", "periodic"])
@pytest.mark.parametrize("X,P,batch", [(64, 8, 2), (64, 32, 2), (100, 16, 2), (128, 32, 2), (180, 8, 2),
                                       (180, 32, 2), (256, 16, 2), (256, 32, 8), (256, 32, 9), (360, 8, 2),
                                       (360, 16, 2), (360, 32, 24), (360, 32, 25)])
def test_whole_iterations_equal_steps_bitwise(otdyn, X, P, batch, per):  # noqa: F811
    print(f"whole iterations {X}x{P} x{batch} per={per}", flush=True)
    for x, y in zip(_run(otdyn, X, P, per, 21, False, batch), _run(otdyn, X, P, per, 21, True, batch)):
        np.testing.assert_array_equal(x, y)


@pytest.mark.parametrize("n,T,count", [(180, 16, 5), (100, 8, 5), (360, 32, 26)])
def test_frozen_members_of_a_group(otdyn, n, T, count):  # noqa: F811
    import torch
    print(f"frozen members {n}x{T} x{count}", flush=True)
    probs = hue_problems(count, seed=21, bins=(n,), steps=(T,))
    d = periodic_desc(otdyn, base_refine=3)
    bt = otdyn.Batch(d, [(n, 1, 1, T)] * count)
    bt.set_boundary([p[2].reshape(1, 1, -1) for p in probs], [p[3].reshape(1, 1, -1) for p in probs])
    status, rep = bt.solve(60000, chunk=100)
    assert status == otdyn.OT_OK
    its = [bt.problem(i).iterations for i in range(count)]
    assert len(set(its)) > 1, its              # frozen at different checks
    for i in sorted({int(np.argmin(its)), int(np.argmax(its)), count // 2}):
        s = periodic_desc(otdyn, base_refine=3)
        s.X, s.Y, s.C, s.P = n, 1, 1, T
        prob = otdyn.Problem(s, "cuda")
        prob.set_boundary(*(torch.from_numpy(probs[i][q].reshape(1, 1, -1)) for q in (2, 3)))
        prob.init()
        prob.step(its[i])
        torch.cuda.synchronize()
        for u, v in zip(bt.state(i), [t[0].cpu().numpy() for t in prob.state()]):
            np.testing.assert_array_equal(u, v)
        prob.close()
    bt.close()
