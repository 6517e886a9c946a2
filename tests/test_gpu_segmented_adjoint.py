"""The segmented adjoint (calls of at most one or two work items per compute unit: the list of an
item in 8 or 2 segments walked side by side) against the FP64 oracle: item counts on both sides of
its limits (256 and 512 items on 256 compute units), list lengths at the edges of a 64-Gaussian batch
and of the segments (one batch, fewer batches than segments, a remainder), cameras, lidars and both
in one call, and the channel buckets it takes; 20 channels and 513 lidar tiles take the general walk.  The upstream
gradient is nonzero on sampled rays only, whose exact gradient the oracle evaluates; the bar is
test_gpu_parity's 1e-3 per element and per tensor."""
import numpy as np
import pytest
import torch

from oracle import grad as ogr
from oracle import render as rd
from scenes import synthetic as S
from tests.gpu_helpers import assert_grad_close

pytestmark = pytest.mark.gpu


def _scene(rng, n, n_feat):
    """A dim cluster ahead: every ray through it blends most of its n Gaussians."""
    mu = rng.normal(size=(n, 3)) * np.array([1.5, 0.5, 0.3]) + np.array([9.0, 0.0, 0.0])
    g = S.random_gaussians(rng, mu, n_feat, rgb=False, moving_frac=0.5)
    g.opacities[:] = rng.uniform(0.01, 0.05, size=n).astype(np.float32)
    return g


def _sensors(kind, tiles, n_ch):
    cams, lids = [], []
    ego = (8.0, 0.0, 0.0)
    if kind in ("camera", "rig"):
        # tiles of 16 x 16 pixels in two rows (one tile: a single row); the cluster spans the centre
        w, h = (16, 16) if tiles == 1 else (16 * (tiles // 2) - 5, 32)
        if tiles % 2 and tiles > 1:
            w, h = 16 * tiles - 5, 16
        cams.append(S.make_camera((0, 0, 0), 0.0, w, h, 60.0, t_rs=0.02, ego_vel_world=ego, n_channels=n_ch))
    if kind in ("lidar", "rig"):
        m = tiles if kind == "lidar" else 16
        lids.append(S.make_lidar((0, 0, 0), 0.0, 8, -8.0, 6.0, 32 * m, ego_vel_world=ego, n_channels=min(n_ch, 8)))
    return cams, lids


@pytest.mark.parametrize("kind,tiles,n,n_ch", [
    ("camera", 1, 1, 3), ("camera", 1, 64, 16), ("camera", 4, 65, 8), ("camera", 255, 520, 16),
    ("camera", 256, 130, 13), ("camera", 257, 700, 16), ("camera", 512, 520, 4),
    ("lidar", 2, 64, 8), ("lidar", 256, 577, 4), ("lidar", 300, 200, 8), ("lidar", 513, 70, 8),
    ("rig", 64, 520, 16), ("rig", 400, 130, 8), ("camera", 32, 200, 20)])
def test_segmented_adjoint(kind, tiles, n, n_ch):
    from paper_2411_16816_amd import binding as b
    b.load()
    rng = np.random.default_rng(1000 * tiles + n)
    print(f"[segments] {kind} tiles {tiles} n {n} channels {n_ch}", flush=True)
    g = _scene(rng, n, max(n_ch, 8))
    cams, lids = _sensors(kind, tiles, n_ch)
    rig = b.Rig(cams, lids)
    G = b.GaussTensors.from_numpy(g)
    sp = b.SensorPass(rig, 0, len(rig.sensors), n, 1, batched=kind == "rig")
    sp.fit_capacity(G)
    sp.render(G)
    dF, dD, dA = np.zeros(sp.n_feat, np.float32), np.zeros(sp.n_rays, np.float32), np.zeros(sp.n_rays, np.float32)
    ref = None
    for k, s in enumerate(rig.sensors):
        rs, fs, C = sp.sensor_slices(k)
        # rays near the cluster (the image's middle columns; azimuth 0 of the lidar) and anywhere
        if k < len(cams):
            col = np.clip(s.width // 2 + rng.integers(-30, 31, 24), 0, s.width - 1)
            idx = np.unique(rng.integers(0, s.height, 24) * s.width + col)
        else:
            col = rng.integers(-40, 41, 24) % s.n_az
            idx = np.unique(rng.integers(0, s.n_beams, 24) * s.n_az + col)
        keep = idx[~rd.render_sensor(g, s, idx)["near"]]   # no decision within rounding
        assert len(keep) >= 0.6 * len(idx)
        uF, uD, uA = S.upstream_grads(tiles + k, len(keep), C)
        dF[fs.start:fs.stop].reshape(-1, C)[keep] = uF
        dD[rs.start + keep], dA[rs.start + keep] = uD, uA
        r, _ = ogr.reference_grads(g, s, keep, uF, uD, uA)
        ref = r if ref is None else {q: ref[q] + r[q] for q in ref}
    grads = b.zeros_like_grads(G)
    t = lambda a: torch.from_numpy(a).cuda()
    sp.raster_bwd(G, t(dF), t(dD), t(dA), grads)
    torch.cuda.synchronize()
    for q in ref:
        # (the one Gaussian of the smallest case may miss every sampled ray)
        assert_grad_close(getattr(grads, q).cpu().numpy(), ref[q], f"{kind} {tiles} {n}: {q}", require_nonzero=n > 1)
