"""The strict order of the pixels at the edges of the device's radix sort (tiles
of 8192 pixels, 64 a round, dealt to eight XCDs): output bins and bytes equal the
oracle's, which depend on every rank."""
import numpy as np
import pytest

from oracle import hue as ref
from synth import inputs
from test_gpu_hue import _frame_check, _renderer, othue  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["random", "few", "one"])
@pytest.mark.parametrize("npix", [63, 8191, 8192, 8193, 9 * 8192 + 1, 17 * 8192 - 3])
def test_order_at_tile_edges(othue, npix, kind):  # noqa: F811
    print(f"hue order {npix} {kind}", flush=True)
    rng = np.random.default_rng(npix)
    img = rng.integers(0, 256, size=(1, npix, 3), dtype=np.uint8)
    if kind == "few":                       # long runs of equal hues
        img = img[:, rng.integers(0, min(npix, 5), size=npix)]
    elif kind == "one":                     # every pixel ties
        img[:] = 77
    r = _renderer(othue, img, 256)
    src = ref.Source(img, 256)
    _frame_check(r, src, inputs.von_mises_hist(npix, 256))
    r.close()
