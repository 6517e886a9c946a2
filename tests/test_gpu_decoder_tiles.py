"""The lidar decoder where its tiles can go wrong: feature counts at the edges of the operands (pairs of
inputs, 16-column tiles, the 8 / 16 / 32 variants), ray counts around the wavefront and the workgroup,
and rows that are not 16-byte aligned, against the FP64 oracle with the bars of test_gpu_decoder.py
(FP32 arithmetic over at most 35 terms and sums over rays stays two orders below); and an infinite or NaN
feature, which reaches the outputs of its own ray only."""
import numpy as np
import pytest
import torch

from test_gpu_decoder import _binding, _close, _dev, _oracle, _rel, _run, _weights

pytestmark = pytest.mark.gpu


def _inputs(n, C, seed):
    rng = np.random.default_rng(seed)
    f = np.float32
    return (rng.normal(size=(n, C)).astype(f), rng.uniform(0, 2 * np.pi, n).astype(f), rng.uniform(-0.45, 0.27, n).astype(f),
            _weights(rng, C), rng.normal(size=n).astype(f), rng.normal(size=n).astype(f))


def _decided(F, az, el, W):
    """Rays whose ReLU decisions a sum in FP32 cannot change: every pre-activation is further from zero
    than (C + 4) roundings of its terms' magnitudes (the direction's own rounding included)."""
    a, e = az.astype(np.float64), el.astype(np.float64)
    x = np.concatenate([F, np.stack([np.cos(e) * np.cos(a), np.cos(e) * np.sin(a), np.sin(e)], 1)], 1)
    w, b1 = W[0].astype(np.float64), W[1].astype(np.float64)
    bound = (F.shape[1] + 4) * 2.0 ** -23 * (np.abs(x) @ np.abs(w).T + np.abs(b1))
    return (np.abs(x @ w.T + b1) > bound).all(1)


@pytest.mark.parametrize("n,C", [(65, 0), (64, 1), (129, 2), (1000, 7), (63, 8), (2049, 9), (127, 15), (1, 16),
                                 (129, 17), (64, 31), (200001, 32), (200001, 5)])
def test_tile_edges(n, C):
    x = _inputs(n, C, 31 * n + C)
    decided = _decided(*x[:4])
    assert decided.mean() > 0.99
    for u in x[4:]:
        u[~decided] = 0     # undecided rays bring no gradient
    I, P, dF, g = _run(_binding(), *x)
    ref = _oracle(*x)
    _close(I, ref[0], "intensity")
    _close(P, ref[1], "drop")
    if C:
        _close(dF, ref[2], "d_feat")
    for f in ("w1", "b1", "w2", "b2"):
        _rel(g[f], ref[3][f], f)


@pytest.mark.parametrize("C", [8, 16, 32])
def test_unaligned_rows(C):
    b = _binding()
    n = 1000
    F, az, el, W, dI, dP = _inputs(n, C, C)
    mlp = b.LidarMLP(*(_dev(w) for w in W))
    Fd = torch.empty(n * C + 1, device="cuda")[1:].view(n, C)   # 4 bytes past a 16-byte boundary
    Fd.copy_(_dev(F))
    dF = torch.zeros(n * C + 1, device="cuda")[1:].view(n, C)
    I, P = b.lidar_decode(Fd, _dev(az), _dev(el), mlp)
    b.lidar_decode_bwd(Fd, _dev(az), _dev(el), mlp, _dev(dI), _dev(dP), dF, {})
    torch.cuda.synchronize()
    ref = _oracle(F, az, el, W, dI, dP)
    _close(I.cpu().numpy(), ref[0], "intensity")
    _close(P.cpu().numpy(), ref[1], "drop")
    _close(dF.cpu().numpy(), ref[2], "d_feat")


@pytest.mark.parametrize("C", [3, 8, 16])
def test_non_finite_features_stay_in_their_ray(C):
    b = _binding()
    F, az, el, W, _, _ = _inputs(300, C, 9)
    W[0] = np.abs(W[0])     # every hidden unit and output grows with the feature
    W[2] = np.abs(W[2])
    F[70, 0], F[131, C - 1] = np.inf, np.nan
    mlp = b.LidarMLP(*(_dev(w) for w in W))
    I, P = b.lidar_decode(_dev(F), _dev(az), _dev(el), mlp)
    ok = np.ones(300, bool)
    ok[[70, 131]] = False
    ref = _oracle(F[ok], az[ok], el[ok], W, az[ok] * 0, az[ok] * 0)
    _close(I.cpu().numpy()[ok], ref[0], "intensity")
    _close(P.cpu().numpy()[ok], ref[1], "drop")
    assert float(I[70]) == 1.0 and float(P[70]) == 1.0                  # sigmoid(+inf)
    b2 = 1.0 / (1.0 + np.exp(-W[3].astype(np.float64)))                 # ReLU(NaN) = 0
    assert abs(float(I[131]) - b2[0]) < 1e-6 and abs(float(P[131]) - b2[1]) < 1e-6
