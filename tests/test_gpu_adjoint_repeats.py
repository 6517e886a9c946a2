"""The adjoint's sums have a fixed order where no two work items add to the same Gaussian's row: the same
call repeated gives the same bits, in every form of the walk (one item per compute unit, two, and more:
8 segments of two wavefronts, 2 segments of four, one walk of two)."""
import numpy as np
import pytest
import torch

from oracle import geometry as geo
from scenes import synthetic as S

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind,size", [("camera", (320, 180)), ("camera", (480, 270)), ("camera", (640, 270)),
                                       ("lidar", (32, 1024)), ("lidar", (128, 1024)), ("lidar", (128, 1280)),
                                       ("rig", (320, 180))])
def test_same_call_same_bits(kind, size):
    from paper_2411_16816_amd import binding as b
    b.load()
    rng = np.random.default_rng(61)
    n = 4000
    mu = np.stack([rng.uniform(-20, 20, n), rng.uniform(-20, 20, n), rng.uniform(-2, 2, n)], 1)
    g = S.random_gaussians(rng, mu, 19, rgb=True, moving_frac=0.4, log_scale_mean=-0.6)
    cams = [] if kind == "lidar" else [S.make_camera((0, 0, 0), 0.0, *size, 0.8 * size[0], t_rs=0.03,
                                                     ego_vel_world=(6.0, 0, 0), n_channels=16)]
    beams, az = (32, 1024) if kind == "rig" else size
    lids = [] if kind == "camera" else [S.make_lidar((0, 0, 0), 0.0, beams, -20.0, 15.0, az, tile_az=32, tile_el=8,
                                                     ego_vel_world=(6.0, 0, 0), feat_offset=3, n_channels=8)]
    print(f"[repeats] {kind} {size}", flush=True)
    rig = b.Rig(cams, lids)
    G = b.GaussTensors.from_numpy(g)
    sp = b.SensorPass(rig, 0, len(rig.sensors), n, 1, batched=kind == "rig")
    sp.fit_capacity(G)
    sp.render(G)
    up = np.random.default_rng(62)
    ups = [torch.from_numpy(up.normal(size=m).astype(np.float32)).cuda() for m in (sp.n_feat, sp.n_rays, sp.n_rays)]
    first = None
    for _ in range(8):
        grads = b.zeros_like_grads(G)
        sp.raster_bwd(G, *ups, grads)
        torch.cuda.synchronize()
        got = {q: getattr(grads, q).cpu().numpy() for q in geo.Params.names}
        first = first or got
        for q in got:
            assert np.abs(first[q]).max() > 0
            assert np.array_equal(got[q], first[q]), (q, int((got[q] != first[q]).sum()))
