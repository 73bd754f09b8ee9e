"""Frames rendered together at the edges of the pixel pass: bins around each
padded power of two, frame counts around the group of a block, and an output
that only the pixel-by-pixel path can write; bins and bytes equal the oracle's."""
import numpy as np
import pytest

from oracle import hue as ref
from synth import inputs
from test_gpu_hue import othue  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [2, 3, 8, 9, 1024, 1025, 2048, 2049, 4096])
@pytest.mark.parametrize("F,npix", [(1, 4096), (2, 4100), (5, 4100), (9, 4101)])
def test_frames_at_the_edges(othue, n, F, npix):  # noqa: F811
    import torch
    print(f"hue frames n={n} F={F} npix={npix}", flush=True)
    rng = np.random.default_rng(n + F)
    img = rng.integers(0, 256, size=(1, npix, 3), dtype=np.uint8)
    img[:, ::7] = img[:, ::7, :1]                   # greys
    img[:, 1::7, 0] = 255                           # reds, where the hue wraps
    src = ref.Source(img, n)
    targets = np.stack([np.roll(inputs.von_mises_hist(n + f, n), f * (n // 3)) for f in range(F)])
    r = othue.HueRenderer(npix, n, max_frames=F)
    r.set_source(torch.from_numpy(img.reshape(-1)).cuda())
    out, bins = r.render_frames(torch.from_numpy(targets.astype(np.float32)).cuda(), with_bins=True)
    for f in range(F):
        rgb_ref, k_ref, _, _ = src.render(targets[f].astype(np.float32))
        assert np.array_equal(bins[f].cpu().numpy().reshape(-1), np.asarray(k_ref).reshape(-1)), f
        assert np.array_equal(out[f].cpu().numpy().reshape(-1), np.asarray(rgb_ref).reshape(-1)), f
    r.close()
