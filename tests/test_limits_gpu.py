"""Calls at the limits of what the library accepts."""
import numpy as np
import pytest

from test_parity_gpu import B, _built  # noqa: F401

pytestmark = pytest.mark.gpu


def _noise(W, H, seed):
    return np.random.default_rng(seed).integers(0, 256, size=(H, W, 3)).astype(np.uint8)


def test_static_query_of_as_many_tiles_as_the_scratch_holds():
    # 32768 SIMT tiles in one row; the aligned MFMA tiling has one more
    W, H, r = 2097167, 9, 4
    rgb = _noise(W, H, 1)
    mask = np.zeros((H, W), np.uint8)
    mask[3:6, 1000:1004] = 1
    g = B.Inpainter(rgb, mask, r)
    rect = (11, 0, W, H)
    want = g.find_exemplar(1000, 4, r, rect)
    assert g.find_exemplar_static(1000, 4, r, rect) == want
    with pytest.raises(B.InpaintError) as e:
        g.find_exemplar_static(1000, 4, r, (10, 0, W, H))
    assert e.value.status == B.INVALID_ARGUMENT
    g.close()
