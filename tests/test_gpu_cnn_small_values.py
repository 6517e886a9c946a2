"""The camera decoder's adjoint on operands near the small end of FP32, about 1e-36: its bf16 parts must
not lose the bits that an FP32 value of that size has.  The upstream gradient (the gradients of every
layer), the stem's weights (the gradient of the features that only the stem reads) and the features (the
gradient of the stem's weights to them) are scaled by 2^-120 in turn.  Against the FP64 oracle with the
bars of test_gpu_cnn.py: FP32 values and sums of this size are multiples of 2^-149, 1e-9 of them, so that
the bars leave the arithmetic the room that they leave it at one."""
import numpy as np
import pytest

from test_gpu_cnn import _binding, _camera, _f32, _oracle, _rel, _weights
from test_gpu_cnn_tiles import _active, _run

pytestmark = pytest.mark.gpu

UP = 2.0 ** 120   # the compared gradients are brought back to order one


@pytest.mark.parametrize("what", ["upstream", "weights", "features"])
def test_small_operands(what):
    b = _binding()
    w, h = 41, 29
    rng = np.random.default_rng(78)
    print(f"[cnn small] {what}", flush=True)
    cam = _camera(w, h)
    W = _active(_weights(rng, 16, 8))
    F = _f32(rng.normal(size=(h, w, 16)))
    dI = _f32(rng.normal(size=(h, w, 3)))
    if what == "upstream":
        dI = _f32(dI / UP)
    elif what == "weights":
        W["w_in"] = _f32(W["w_in"] / UP)
    else:
        F = _f32(F / UP)
    _, dF, g = _run(b, cam, W, F, dI)
    _, r = _oracle(F, cam, W, dI)
    up = lambda a: np.asarray(a, np.float64) * UP
    if what == "weights":
        _rel(up(dF[..., 3:]), up(r["F"][..., 3:]), "d_feat")
    elif what == "features":
        _rel(up(g["w_in"][:, :16]), up(r["w_in"][:, :16]), "w_in")
    else:
        _rel(up(dF), up(r["F"]), "d_feat")
        for k in ("embed", "w_in", "b_in", "w_out", "b_out"):
            _rel(up(g[k]), up(r[k]), k)
        for j in range(4):
            _rel(up(g["w_block"][j]), up(r["w_block"][j]), f"w_block{j}")
            _rel(up(g["b_block"][j]), up(r["b_block"][j]), f"b_block{j}")
