"""The pixel pass with one and with four frames per block: the same images as a call
of many frames (four per block, the last block fewer) and in calls of fewer frames
(one per block) are equal byte for byte, and single frames of it equal the
oracle's; pixels in groups of four and pixel by pixel."""
import numpy as np
import pytest

from oracle import hue as ref
from test_gpu_hue import othue  # noqa: F401

pytestmark = pytest.mark.gpu


# 2 blocks a frame: four frames per block from 7168 blocks in all (512 bins and fewer) and 28672
# (1024), pixel by pixel from half of that
@pytest.mark.parametrize("n,F,npix", [(12, 3585, 2000), (300, 3587, 2000), (512, 3590, 2003), (600, 16385, 1100),
                                      (700, 7171, 1101)])
def test_many_frames_equal_few(othue, n, F, npix):  # noqa: F811
    import torch
    print(f"hue groups n={n} F={F} npix={npix}", flush=True)
    rng = np.random.default_rng(n)
    img = rng.integers(0, 256, size=(1, npix, 3), dtype=np.uint8)
    img[:, ::5] = img[:, ::5, :1]
    targets = torch.from_numpy((rng.random((F, n), dtype=np.float32) ** 4 + 1e-3)).cuda()
    r = othue.HueRenderer(npix, n, max_frames=F)
    r.set_source(torch.from_numpy(img.reshape(-1)).cuda())
    out, bins = r.render_frames(targets, with_bins=True)
    for a in range(0, F, 1500):
        o, b = r.render_frames(targets[a:a + 1500].contiguous(), with_bins=True)
        assert torch.equal(o, out[a:a + 1500]) and torch.equal(b, bins[a:a + 1500]), a
    src = ref.Source(img, n)
    for f in (0, F // 2, F - 1):
        rgb_ref, k_ref, _, _ = src.render(targets[f].cpu().numpy())
        assert np.array_equal(bins[f].cpu().numpy().reshape(-1), np.asarray(k_ref).reshape(-1)), f
        assert np.array_equal(out[f].cpu().numpy().reshape(-1), np.asarray(rgb_ref).reshape(-1)), f
    r.close()
