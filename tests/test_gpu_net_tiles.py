"""GPU checks of the network's kernels where their tiles end: the layout maps
at pixel and channel counts around a tile of 64, and convolutions on images
smaller than a tile, images that share a tile, channel counts that straddle
the steps of 16 and the unstaged route (channels that do not fit in LDS).

The maps are FP32 sums of at most four terms of magnitude <= 4: 1e-6.  The
network is compared with the FP64 oracle on BF16-rounded inputs and weights;
each of its tensors is rounded to BF16 (2^-9 relative), which compounds over
the layers: 2e-2.
"""
import numpy as np
import pytest

from oracle import nn

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def N():
    import torch
    from paper_1501_04840_amd import otnet
    assert torch.cuda.is_available()
    otnet.lib()
    return otnet


def _bf16(a):
    u = np.ascontiguousarray(a, dtype=np.float32).view(np.uint32).astype(np.uint64)
    u = (u + 0x7FFF + ((u >> 16) & 1)) & 0xFFFF0000
    return u.astype(np.uint32).view(np.float32).astype(np.float64)


# X Y pixels and C (P - 1) + 3 C P channels: below, at and past 64 of each
@pytest.mark.parametrize("X,Y,C,P,nb,with_base", [(3, 5, 1, 2, 1, True), (8, 8, 1, 16, 1, False), (13, 5, 1, 17, 2, True),
                                                  (16, 12, 3, 6, 3, True), (7, 9, 3, 21, 2, True)])
def test_layout_maps_at_tile_edges(N, X, Y, C, P, nb, with_base):
    import torch
    from paper_1501_04840_amd import otdyn
    print(f"maps {X}x{Y}x{C}x{P} x{nb}", flush=True)
    d = otdyn.ot_dyn_default_desc(X, Y, C, P)
    rng = np.random.default_rng(X * Y + P)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a, np.float32)).to("cuda:0")
    f0, f1 = rng.uniform(0, 1, (2, nb, C, Y, X)).astype(np.float32)
    F = rng.standard_normal((nb, P + 1, C, Y, X)).astype(np.float32)
    M = rng.standard_normal((3, nb, P, C, Y, X)).astype(np.float32)
    nch = N.warm_channels(C, P)
    base = rng.standard_normal((nb, Y, X, nch)).astype(np.float32)
    db = dev(base) if with_base else None
    sl = X * Y * C
    st = torch.cuda.current_stream().cuda_stream
    wall = np.ones((3, 1, 1, C, Y, X))
    wall[0, ..., 0] = 0
    wall[1, ..., 0, :] = 0                       # colour: periodic
    if C == 1:
        wall[2] = 1                              # the descriptor's colour axis stays periodic
    s = (np.arange(1, P) / P).reshape(1, P - 1, 1, 1, 1)
    lin = (1 - s) * f0[:, None].astype(float) + s * f1[:, None]
    chan = lambda v: np.moveaxis(v.reshape(nb, -1, Y, X), 1, -1)
    b0 = base if with_base else np.zeros_like(base)
    keep = np.concatenate([np.ones((nb, Y, X, C * (P - 1)))] +
                          [chan(np.broadcast_to(wall[q], (nb, P, C, Y, X)).copy()) for q in range(3)], -1)
    ref = (np.concatenate([chan(F[:, 1:P] - lin)] + [chan(M[q].astype(float)) for q in range(3)], -1) - b0) * keep
    t = torch.full((nb, Y, X, nch), 7.0, device="cuda:0")
    N.ot_warm_targets(d, nb, dev(f0), dev(f1), dev(F), (P + 1) * sl, *(dev(m) for m in M), P * sl, db, t, st)
    np.testing.assert_allclose(t.cpu().numpy(), ref, rtol=0, atol=1e-6)
    x = torch.empty((nb, Y, X, 2 * C + (nch if with_base else 0)), device="cuda:0")
    N.ot_warm_inputs(d, nb, dev(f0), dev(f1), db, x, st)
    want = np.concatenate([np.moveaxis(f0, 1, -1), np.moveaxis(f1, 1, -1)] + ([base] if with_base else []), -1)
    np.testing.assert_array_equal(x.cpu().numpy(), want)
    y = rng.standard_normal((nb, Y, X, nch)).astype(np.float32)
    F2 = torch.zeros((nb, P + 1, C, Y, X), device="cuda:0")
    M2 = torch.full((3, nb, P, C, Y, X), 7.0, device="cuda:0")
    N.ot_warm_state(d, nb, dev(f0), dev(f1), dev(y), db, F2, (P + 1) * sl, *M2, P * sl, st)
    back = np.moveaxis((y + b0) * keep, -1, 1)
    np.testing.assert_allclose(F2.cpu().numpy()[:, 1:P], lin + back[:, :C * (P - 1)].reshape(nb, P - 1, C, Y, X), rtol=0, atol=1e-6)
    got = back[:, C * (P - 1):].reshape(nb, 3, P, C, Y, X)
    np.testing.assert_allclose(M2.cpu().numpy(), np.moveaxis(got, 1, 0), rtol=0, atol=1e-6)


# H, W, in, out, base, levels, batch: images smaller than the 8 x 8 tile and
# sharing it (an odd count of them), tiles cut by the image, 8 channels (a step
# spans two taps), 24 and 104 channels (steps straddle taps), one fragment and
# many, outputs past a fragment, and more channels than a staged tile holds
NETS = [
    (4, 4, 3, 5, 8, 2, 5),
    (2, 6, 8, 9, 8, 1, 3),
    (12, 20, 20, 40, 24, 2, 2),
    (16, 8, 100, 70, 16, 3, 3),
    (24, 24, 35, 33, 40, 2, 9),
    (8, 8, 1000, 8, 8, 1, 1),
]


@pytest.mark.parametrize("case", NETS, ids=lambda c: "x".join(map(str, c)))
def test_convolution_tiles_match_oracle(N, case):
    import torch
    H, W, cin, cout, base, levels, nb = case
    print(f"net {case}", flush=True)
    d = N.ot_net_default_desc(64, 64, cin, cout, nb)      # (checks its sizes for four levels)
    d.H, d.W, d.base, d.levels = H, W, base, levels
    specs = nn.layer_specs(cin, cout, base, levels)
    rng = np.random.default_rng(cin + cout)
    flat = nn.he_init(specs, 5) + 0.02 * rng.standard_normal(nn.param_count(specs))
    params = nn.unflatten(specs, flat)
    flat = np.concatenate([np.concatenate([_bf16(Wt).ravel(), np.float32(b).astype(np.float64)])
                           for Wt, b in (params[s[0]] for s in specs)])
    params = nn.unflatten(specs, flat)
    x = _bf16(rng.uniform(0.0, 2.0, size=(nb, H, W, cin)))
    t = rng.standard_normal((nb, H, W, cout))
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a, np.float32)).to("cuda:0")
    net = N.Net(d, "cuda:0")
    net.set_params(dev(flat))
    rel = lambda a, b: float(np.linalg.norm(a - b) / np.linalg.norm(b))
    y = net.forward(dev(x)).cpu().numpy()
    assert rel(y, nn.forward(specs, params, x, levels)) < 2e-2
    y1 = net.forward(dev(x[:1])).cpu().numpy()       # a smaller batch through the same net
    np.testing.assert_array_equal(y1[0], y[0])
    loss, g = net.grad(dev(x), dev(t), dev(np.ones(cout) / cout))
    L, grads = nn.backward(specs, params, x, t, [(c, c + 1, 1.0 / cout) for c in range(cout)], levels)
    assert abs(loss - L) <= 2e-2 * abs(L)
    g, gr = g.cpu().numpy().astype(np.float64), nn.flatten_grads(specs, grads)
    assert g @ gr / (np.linalg.norm(g) * np.linalg.norm(gr)) > 0.999
    net.close()
