"""The camera decoder with several tiles to each persistent workgroup: 480 x 480 pixels make 900
convolution tiles and 1800 weight-gradient tiles for 256 workgroups, so that the input gradient's two
register sets are loaded ahead, staged and loaded again, up to a fourth tile.  Image and gradients against
the FP64 oracle: gradients with the bars of test_gpu_cnn.py, the image with its bar scaled to the image's
magnitude (the biases that keep every ReLU's input away from zero make values of about 200)."""
import numpy as np
import pytest

from test_gpu_cnn import _binding, _camera, _f32, _oracle, _weights
from test_gpu_cnn_tiles import _active, _check, _run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("w,h", [(272, 272), (480, 480)])
def test_many_tiles(w, h):
    b = _binding()
    rng = np.random.default_rng(w + 3 * h)
    print(f"[cnn many tiles] {w}x{h}", flush=True)
    cam = _camera(w, h)
    W = _active(_weights(rng, 16, 8))
    F = _f32(rng.normal(size=(h, w, 16)))
    dI = _f32(rng.normal(size=(h, w, 3)))
    I, dF, g = _run(b, cam, W, F, dI)
    ref, r = _oracle(F, cam, W, dI)
    _check(I, dF, g, ref, r, image=False)
    bad = np.abs(I - ref) > 1e-4 * np.abs(ref) + 1e-5 * np.abs(ref).max()
    assert not bad.any(), (int(bad.sum()), float(np.abs(I - ref).max()), float(np.abs(ref).max()))


def test_large_values_in_later_tiles():
    """Two upstream values of 3e30, whose products do not fit the scaled bf16 parts' range, in the third and
    the fourth tile of their workgroups: those outputs and weight sums are contracted again, and nothing
    outside the network's reach changes."""
    b = _binding()
    w, h = 480, 480
    rng = np.random.default_rng(15)
    print("[cnn many tiles] large values", flush=True)
    cam = _camera(w, h)
    W = _active(_weights(rng, 16, 8))
    F = _f32(rng.normal(size=(h, w, 16)))
    dI = _f32(rng.normal(size=(h, w, 3)))
    clean = _run(b, cam, W, F, dI)
    far = np.ones((h, w), bool)
    for y, x in ((300, 33), (470, 477)):   # convolution tiles 542 and 899 of 900
        dI[y, x, 1] = 3.0e30
        far[y - 5:y + 6, x - 5:x + 6] = False
    I, dF, g = _run(b, cam, W, F, dI)
    assert np.array_equal(I, clean[0]) and np.array_equal(dF[far], clean[1][far])
    _check(I, dF, g, *_oracle(F, cam, W, dI), image=False)
