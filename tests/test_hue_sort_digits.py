"""The device's strict order sorts pixels by the 19-bit key floor(h 2^19) of
their FP32 hue in two digits, of 9 and 10 bits: the key is strictly increasing
across the distinct hues of 8-bit RGB."""
import numpy as np

from oracle import hue


def test_19_bit_key_orders_all_8_bit_hues_like_the_hue():
    v = np.arange(256, dtype=np.uint8)
    hs = []
    for r0 in range(256):
        g, b = np.meshgrid(v, v, indexing="ij")
        px = np.stack([np.full(65536, r0, np.uint8), g.ravel(), b.ravel()], axis=-1)
        hs.append(np.unique(hue.hue_of_rgb(px)[0]))
    h = np.unique(np.concatenate(hs))                       # every attainable FP32 hue
    key = np.floor(h.astype(np.float64) * 2.0 ** 19)        # exact: power-of-two scaling
    assert np.all(np.diff(key) > 0)
    assert key.min() >= 0 and key.max() < 2 ** 19
