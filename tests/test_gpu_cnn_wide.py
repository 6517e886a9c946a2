"""The camera decoder on an image wider than the buffer windows address and with pixels past 2^31 bytes:
900001 x 20, features and upstream gradients in its left and right ends.  Against the FP64 oracle on the
two ends (the network reaches 5 pixels, so a crop with that margin is exact), with the bars of
test_gpu_cnn.py."""
import dataclasses

import numpy as np
import pytest

from test_gpu_cnn import _binding, _camera, _close, _f32, _oracle, _rel, _weights
from test_gpu_cnn_tiles import _run

pytestmark = pytest.mark.gpu


def test_wide_image_at_both_ends():
    b = _binding()
    w, h, m = 900001, 20, 24
    rng = np.random.default_rng(9)
    print(f"[cnn wide] {w}x{h}", flush=True)
    cam = dataclasses.replace(_camera(w, h), cx=450000.0, fx=4.0e5, fy=4.0e5)
    W = _weights(rng, 16, 8)
    F = np.zeros((h, w, 16), np.float32)
    dI = np.zeros((h, w, 3), np.float32)
    ends = [(slice(0, m + 5), slice(0, m), slice(0, m - 5)), (slice(w - m - 5, w), slice(w - m, w), slice(w - m + 5, w))]
    for crop, _, up in ends:
        F[:, crop] = rng.normal(size=(h, m + 5, 16))
        dI[:, up] = rng.normal(size=(h, m - 5, 3))
    I, dF, g = _run(b, cam, W, F, dI)
    assert (dF[:, m + 5:w - m - 5] == 0).all()
    total = None
    for crop, exact, _ in ends:
        c = dataclasses.replace(cam, width=m + 5, cx=cam.cx - crop.start)
        ref, r = _oracle(F[:, crop], c, W, dI[:, crop])
        inner = slice(exact.start - crop.start, exact.stop - crop.start)
        _close(I[:, exact], ref[:, inner], "image")
        _rel(dF[:, crop], r["F"], "d_feat")
        flat = {q: r[q] for q in ("embed", "w_in", "b_in", "w_out", "b_out")}
        flat.update({f"{q}{j}": r[q][j] for q in ("w_block", "b_block") for j in range(4)})
        total = flat if total is None else {q: total[q] + flat[q] for q in flat}
    for q in total:
        _rel(g[q] if q in g else g[q[:-1]][int(q[-1])], total[q], q)
