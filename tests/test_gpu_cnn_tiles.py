"""The camera decoder's convolutions where their tiles and operand splits can go wrong: images at the
edges of the 16 x 16 and 8 x 16 tiles, more tiles than workgroups, values that do not split into bf16
parts (infinities, NaN) or span the type's range, and an image wider than the buffer
windows address.  Against the FP64 oracle with the bars of test_gpu_cnn.py (1e-4 of the norm: FP32
arithmetic over contractions of 288 terms and sums over pixels stays two orders below)."""
import dataclasses

import numpy as np
import pytest
import torch

from oracle import decoders as dec
from test_gpu_cnn import _binding, _camera, _close, _dev_cnn, _f32, _oracle, _rel, _weights

pytestmark = pytest.mark.gpu


def _run(b, cam, W, F, dI):
    cnn = _dev_cnn(b, W)
    ws = b.camera_decode_workspace(cam)
    Fd = torch.from_numpy(F.reshape(-1)).cuda()
    I = b.camera_decode(cam, Fd, cnn, ws)
    z = torch.zeros_like
    dF = z(Fd)
    g = {"embed": z(cnn.embed), "w_in": z(cnn.w_in), "b_in": z(cnn.b_in), "w_block": [z(x) for x in cnn.w_block],
         "b_block": [z(x) for x in cnn.b_block], "w_out": z(cnn.w_out), "b_out": z(cnn.b_out)}
    b.camera_decode_bwd(cam, Fd, cnn, torch.from_numpy(dI.reshape(-1)).cuda(), dF, g, ws)
    torch.cuda.synchronize()
    n = lambda t: t.cpu().numpy()
    g = {k: [n(x) for x in v] if isinstance(v, list) else n(v) for k, v in g.items()}
    return n(I).reshape(dI.shape), n(dF).reshape(F.shape), g


def _check(I, dF, g, ref, r, image=True):
    if image:
        _close(I, ref, "image")
    _rel(dF, r["F"], "d_feat")
    for k in ("embed", "w_in", "b_in", "w_out", "b_out"):
        _rel(g[k], r[k], k)
    for j in range(4):
        _rel(g["w_block"][j], r["w_block"][j], f"w_block{j}")
        _rel(g["b_block"][j], r["b_block"][j], f"b_block{j}")


def _active(W):
    """Biases that keep the ReLUs' inputs away from zero: no sign decision within rounding."""
    W["b_in"] = W["b_in"] + 10.0
    W["b_block"] = [x + 20.0 for x in W["b_block"]]
    return W


@pytest.mark.parametrize("w,h", [(15, 7), (16, 8), (17, 9), (33, 1), (1, 33), (48, 16), (272, 272)])
def test_tile_edges(w, h):
    # 272 x 272: 289 convolution tiles and 578 weight-gradient tiles for 256 persistent workgroups
    b = _binding()
    rng = np.random.default_rng(1000 * w + h)
    print(f"[cnn tiles] {w}x{h}", flush=True)
    cam = _camera(w, h)
    W = _weights(rng, 16, 8)
    large = w * h > 10000
    if large:   # no ReLU decision near zero; the image, of values about 200, is not the subject here
        W = _active(W)
    F = _f32(rng.normal(size=(h, w, 16)))
    dI = _f32(rng.normal(size=(h, w, 3)))
    _check(*_run(b, cam, W, F, dI), *_oracle(F, cam, W, dI), image=not large)


@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan, 3.0e33])
def test_upstream_that_does_not_split(value):
    """One pixel's upstream gradient is not finite, or 33 orders above the others (its products with
    the activations of about 100 and the weights stay in range)."""
    b = _binding()
    w, h = 41, 29
    rng = np.random.default_rng(77)
    print(f"[cnn tiles] upstream {value}", flush=True)
    cam = _camera(w, h)
    W = _active(_weights(rng, 16, 8))
    F = _f32(rng.normal(size=(h, w, 16)))
    dI = _f32(rng.normal(size=(h, w, 3)))
    clean = _run(b, cam, W, F, dI)
    dI[14, 20, 1] = value
    I, dF, g = _run(b, cam, W, F, dI)
    assert np.array_equal(I, clean[0])
    far = np.ones((h, w), bool)     # outside the five convolutions' reach nothing changes
    far[9:20, 15:26] = False
    assert np.array_equal(dF[far], clean[1][far])
    if np.isfinite(value):
        _check(I, dF, g, *_oracle(F, cam, W, dI), image=False)
        return
    assert not np.isfinite(dF[9:20, 15:26]).any()
    # the last convolution's output gradient at the pixel is value (w_out[1] f + w_out[4]) where its
    # ReLU is on; a weight's gradient there is that times the convolution's input
    t = lambda a: torch.from_numpy(np.asarray(_f32(a), np.float64))
    x = torch.cat([t(F), dec.camera_directions(cam), t(W["embed"]).expand(h, w, 8)], -1)
    hid = torch.relu(dec.conv3x3(x, t(W["w_in"]), t(W["b_in"])))
    for k in range(2):
        r = torch.relu(dec.conv3x3(hid, t(W["w_block"][2 * k]), t(W["b_block"][2 * k])))
        hid = torch.relu(hid + dec.conv3x3(r, t(W["w_block"][2 * k + 1]), t(W["b_block"][2 * k + 1])))
    Wo = _f32(W["w_out"])
    with np.errstate(invalid="ignore"):
        up = np.where(hid[14, 20].numpy() > 0, Wo[1] * (np.float32(value) * F[14, 20, 1]) + Wo[4] * np.float32(value), 0)
        want = up[:, None, None, None] * r[13:16, 19:22].permute(2, 0, 1).numpy()[None]
    for a, e in ((g["b_block"][3], up), (g["w_block"][3], want)):
        assert np.array_equal(np.isfinite(a), np.isfinite(e))
        bad = ~np.isfinite(e)
        assert bad.any() and np.array_equal(a[bad].astype(np.float64), e[bad], equal_nan=True)


def test_image_wider_than_the_windows():
    b = _binding()
    w, h, m = 900001, 1, 24
    rng = np.random.default_rng(5)
    print(f"[cnn tiles] {w}x{h}", flush=True)
    cam = dataclasses.replace(_camera(w, h), cx=12.0, fx=300.0, fy=300.0)
    W = _weights(rng, 16, 8)
    F = np.zeros((h, w, 16), np.float32)
    F[:, :m + 5] = rng.normal(size=(h, m + 5, 16))
    dI = np.zeros((h, w, 3), np.float32)
    dI[:, :m - 5] = rng.normal(size=(h, m - 5, 3))
    I, dF, g = _run(b, cam, W, F, dI)
    crop = dataclasses.replace(cam, width=m + 5)
    ref, r = _oracle(F[:, :m + 5], crop, W, dI[:, :m + 5])
    assert (dF[:, m + 5:] == 0).all()
    _check(I[:, :m], dF[:, :m + 5], g, ref[:, :m], r)
