"""The adjoint's general walk (calls of more than two work items per compute unit, which the segmented
form leaves to it) against the FP64 oracle, in each kernel that runs it: one camera, one lidar, the
persistent queue of cameras only, of lidars only, of both grouped by kind, and of both in one cost order
(without per-entry rows, and with rows on lists that were binned without).  Each with what a call can ask
of the walk: the line-of-sight gradient, the camera's time offset and velocities, lidar tiles split over
two items, tiles of one item, and a capped lidar whose dropped rays carry an upstream gradient that must
be ignored; and the captured step against eager calls.  The upstream gradient is otherwise nonzero on
sampled rays only, whose exact gradient the oracle evaluates; the bar is test_gpu_parity's 1e-3 per
element and per tensor."""
import numpy as np
import pytest
import torch

from oracle import geometry as geo
from oracle import grad as ogr
from oracle import render as rd
from oracle import tiles as ot
from scenes import synthetic as S
from tests.gpu_helpers import assert_grad_close

pytestmark = pytest.mark.gpu


def _binding():
    from paper_2411_16816_amd import binding
    binding.load()
    return binding


def _scene(seed, n=2500):
    """Dim enough that the rays walk most of their lists."""
    rng = np.random.default_rng(seed)
    mu = np.stack([rng.uniform(-14, 14, n), rng.uniform(-14, 14, n), rng.uniform(-1.5, 1.5, n)], 1)
    g = S.random_gaussians(rng, mu, 16, rgb=True, moving_frac=0.4, log_scale_mean=-0.6)
    g.opacities[:] *= np.float32(0.3)
    return g


def _camera(k, w, h):
    cam = S.make_camera((0.2 * k, 0, 0), 40.0 * k, w, h, 0.9 * w, t_rs=0.04, ego_vel_world=(6.0, 0.5, 0),
                        ego_yaw_rate=0.3, n_channels=16)
    cam.time_offset = 0.006
    return cam


def _lidar(k, n_beams, n_az, tile_az, capped=False):
    """Tiles of 8 beams: 16 azimuths make 128 rays, 64 make 512 (two items, or a tile that the cap halves)."""
    lid = S.make_lidar((0, 0.1 * k, 0), 5.0 * k, n_beams, -15.0, 15.0, n_az, tile_az=tile_az, tile_el=8, t_sweep=0.1,
                       ego_vel_world=(10.0, 1.0, 0), ego_yaw_rate=0.2, feat_offset=3, n_channels=8)
    rng = np.random.default_rng(90 + k)
    lid.ray_range = rng.uniform(0.5, 16.0, lid.n_rays).astype(np.float32)
    lid.los_eps = 0.8
    if capped:
        lid.ray_priority = rng.integers(0, 1 << 16, lid.n_rays).astype(np.uint16)
    return lid


def _sensors(form):
    if form == "camera":                                  # 35 x 16 tiles
        return [_camera(0, 560, 250)], []
    if form == "lidar":                                   # 8 x 80 tiles
        return [], [_lidar(0, 64, 1280, 16)]
    if form == "split lidar":                             # 288 tiles of two items each
        return [], [_lidar(0, 64, 2304, 64)]
    if form == "cameras":                                 # 25 x 12 and 23 x 13 tiles
        return [_camera(0, 400, 190), _camera(1, 357, 208)], []
    if form == "lidars":                                  # 256 + 320 tiles; 64 tiles of two items; 32 capped
        return [], [_lidar(0, 32, 1024, 16), _lidar(1, 32, 1280, 16), _lidar(2, 32, 1024, 64), _lidar(3, 16, 1024, 64, True)]
    return ([_camera(0, 400, 190), _camera(1, 250, 110)],  # 300 + 112 tiles, then 128, 64 x 2 and 32 capped
            [_lidar(0, 16, 1024, 16), _lidar(1, 32, 1024, 64), _lidar(2, 16, 1024, 64, True)])


def _assert_general(sp):
    """More items than the segmented form takes."""
    lid = [s for s in sp.rig.sensors if hasattr(s, "ray_az")]
    lidar_tiles = sum(s.n_az_tiles * s.n_el_tiles for s in lid)
    items = sp.n_tiles - lidar_tiles + max(lidar_tiles, -(-sum(s.n_rays for s in lid) // 256))
    assert items > 2 * torch.cuda.get_device_properties(0).multi_processor_count, items


FORMS = ("camera", "lidar", "split lidar", "cameras", "lidars", "rig", "rig without rows", "rig binned without rows")


@pytest.mark.parametrize("form", FORMS)
def test_general_walk(form):
    b = _binding()
    g = _scene(50 + FORMS.index(form))
    cams, lids = _sensors(form)
    print(f"[general walk] {form}", flush=True)
    G = b.GaussTensors.from_numpy(g)
    rig = b.Rig(cams, lids)
    n_s = len(rig.sensors)
    t = lambda a: torch.from_numpy(a).cuda()
    try:
        if form == "rig without rows":
            b.set_adjoint_row_limit(0)
        sp = b.SensorPass(rig, 0, n_s, g.n, 1, batched=n_s > 1)
        sp.fit_capacity(G)
        if form == "rig binned without rows":
            b.set_adjoint_row_limit(0)
        sp.render(G)
        if form == "rig binned without rows":
            b.set_adjoint_row_limit(b.ADJOINT_ROW_LIMIT)
        _assert_general(sp)
        assert int((sp.tile_range[:, 1] - sp.tile_range[:, 0]).max()) > 128   # several batches of 64
        dF = np.zeros(sp.n_feat, np.float32)
        dD, dA, dl = (np.zeros(sp.n_rays, np.float32) for _ in range(3))
        want, want_s = None, []
        for k, s in enumerate(rig.sensors):
            rs, fs, C = sp.sensor_slices(k)
            rng = np.random.default_rng(1000 + k)
            is_lid = k >= len(cams)
            drop = np.zeros(s.n_rays, bool)
            if is_lid and getattr(s, "ray_priority", None) is not None:
                a, e, v = ot.lidar_ray_tiles_f32(s.ray_az, s.ray_el, s)
                drop = ot.lidar_training_dropped(a, e, v, s.ray_priority, s.n_az_tiles, cap=256)
                assert 0.3 < drop.mean() < 0.6
            idx = np.sort(rng.choice(np.nonzero(~drop)[0], 32, replace=False))
            keep = idx[~rd.render_sensor(g, s, idx)["near"]]   # no decision within rounding
            assert len(keep) >= 0.6 * len(idx)
            uF, uD, uA = S.upstream_grads(70 + k, len(keep), C)
            ul = rng.normal(size=len(keep)).astype(np.float32) if is_lid else None
            d = np.nonzero(drop)[0]
            for arr, up in ((dF[fs.start:fs.stop].reshape(-1, C), uF), (dD[rs], uD), (dA[rs], uA), (dl[rs], ul)):
                if up is not None:
                    arr[keep] = up
                    arr[d] = 1.0
            r, _ = ogr.reference_grads(g, s, keep, uF, uD, uA, dlos=ul)
            want = r if want is None else {q: want[q] + r[q] for q in want}
            if not is_lid:
                want_s.append(ogr.reference_sensor_grads(g, s, keep, uF, uD, uA)[0])
        grads = b.zeros_like_grads(G)
        sg = {"sensor_lin_vel": torch.zeros(n_s, 3, device="cuda"), "sensor_ang_vel": torch.zeros(n_s, 3, device="cuda"),
              "sensor_time_offset": torch.zeros(n_s, device="cuda")}
        sp.raster_bwd(G, t(dF), t(dD), t(dA), grads, d_los=t(dl), sensor_grads=sg)
        torch.cuda.synchronize()
    finally:
        b.set_adjoint_row_limit(b.ADJOINT_ROW_LIMIT)
    for q in want:
        assert_grad_close(getattr(grads, q).cpu().numpy(), want[q], f"{form} {q}")
    for k, r in enumerate(want_s):
        for q in r:
            assert_grad_close(sg["sensor_" + q][k].cpu().numpy(), r[q], f"{form} camera {k} {q}")


def test_captured_step():
    """The captured step whose adjoint is the general walk: every replay (the rig moved in between)
    against eager calls, forward bits equal and gradients up to the order of the split tiles' atomics."""
    b = _binding()
    g = _scene(71)
    cams, lids = _sensors("rig")
    rig = b.Rig(cams, lids)
    G = b.GaussTensors.from_numpy(g)
    n_s = len(rig.sensors)
    sp = b.SensorPass(rig, 0, n_s, g.n, 1, batched=True)
    sp.fit_capacity(G, margin=2.0)
    ref = b.SensorPass(rig, 0, n_s, g.n, sp.k_cap, batched=True)
    _assert_general(sp)
    up = np.random.default_rng(7)
    ups = [torch.from_numpy((f * up.normal(size=n)).astype(np.float32)).cuda()
           for f, n in ((1.0, sp.n_feat), (0.1, sp.n_rays), (1.0, sp.n_rays), (1.0, sp.n_rays))]
    gpipe = b.zeros_like_grads(G)
    pipe = b.Pipeline(sp, G, b.BOX, gpipe, *ups[:3], d_los=ups[3])
    for k in range(3):
        print(f"[general walk] replay {k}", flush=True)
        for c in cams:
            c.t = (c.t + np.array([0.0, 0.0, -0.05], np.float32)).astype(np.float32)
        rig.update(cams, lids)
        ref.status.zero_()
        ref.render(G)
        gref = b.zeros_like_grads(G)
        ref.raster_bwd(G, *ups[:3], gref, d_los=ups[3])
        torch.cuda.synchronize()
        pipe.run()
        torch.cuda.synchronize()
        assert b.read_status(sp.status).overflow == 0
        for key in ("feat", "depth", "alpha", "t_final", "last"):
            np.testing.assert_array_equal(sp.outputs()[key].cpu().numpy(), ref.outputs()[key].cpu().numpy(), err_msg=key)
        for q in geo.Params.names:
            x, y = (getattr(z, q).cpu().numpy().astype(np.float64) for z in (gpipe, gref))
            assert np.linalg.norm(y) > 0 and np.linalg.norm(x - y) <= 1e-5 * np.linalg.norm(y), (k, q)
    pipe.close()
