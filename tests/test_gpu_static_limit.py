"""ot_dyn_solve_static at its size limit: problems that fit the library's array
but for the matrices of the dense three-pass solve (a workspace of the caller's
holds those too) are solved, by the same kernels and so bit for bit as with a
workspace of the caller's."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(90, 90, 1, 63), (131, 100, 3, 13), (300, 200, 2, 4)])
def test_static_solve_at_the_limit(shape):
    import torch
    from paper_1501_04840_amd import otdyn
    X, Y, C, P = shape
    print("static solve at the limit", shape, flush=True)
    d = otdyn.ot_dyn_default_desc(X, Y, C, P)
    d.check_every = 8
    excess = otdyn.ot_dyn_workspace_size(d) - otdyn.OT_DYN_STATIC_BYTES
    assert 0 < excess < 1 << 20
    gen = torch.Generator(device="cuda").manual_seed(11)
    f = torch.rand(2, 1, C, Y, X, generator=gen, device="cuda") + 0.5
    f = f / f.mean(dim=(2, 3, 4), keepdim=True)
    f0, f1 = f[0].contiguous(), f[1].contiguous()
    ref = otdyn.Problem(d, "cuda")
    ref.set_boundary(f0, f1)
    ref.init()
    st_ref, rep_ref = ref.solve(16)
    F = torch.full((1, P + 1, C, Y, X), 7.0, device="cuda")
    M = [torch.full((1, P, C, Y, X), -3.0, device="cuda") for _ in range(3)]
    torch.cuda.synchronize()
    stream = torch.cuda.current_stream()
    st, rep = otdyn.ot_dyn_solve_static(d, stream.cuda_stream, f0, f1, F, *M, 16)
    torch.cuda.synchronize()
    assert st == st_ref and rep.iterations == rep_ref.iterations
    for a, b in zip((F, *M), ref.state()):
        assert torch.equal(a, b)
    ref.close()
