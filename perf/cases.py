"""The work that a program has this package do, as cases that can be timed and compared.

A program that trains a scene renders cameras and lidar sweeps of a few thousand to two million
Gaussians forward and backward (one sensor at a time through the per-kind calls or autograd, or a
whole rig as one captured step), decodes the rendered features (lidar MLP, camera CNN) forward and
backward, composes moving actors into the world frame, and now and then regularises and relocates
Gaussians; a program that simulates runs the forward calls alone.  Each of those is a kind of case
(`op`); its sizes run from a handful of thousand rays to full sweeps and 1920 x 1080 images.

    listed()             the cases
    draw(rng)            one more case of the same ranges
    prepare(case, seed)  the inputs and the handles a program keeps
    run(state)           one pass through the public entry points, and its outputs
    work(case)           bytes and operations a pass cannot do without
    exact(case, seed)    the same outputs in 64 bits with plain torch
"""
import math
from types import SimpleNamespace

import numpy as np
import torch

from paper_2411_16816_amd import binding as B

DEV = "cuda"
F64 = torch.float64
PAIRS_PER_RAY = 60      # (ray, Gaussian) pairs a ray blends or tests in these scenes, roughly
EXACT_PAIRS = 4.0e8     # rays x Gaussians up to which the 64-bit render is quick


def listed():
    return [
        # one plain lidar sweep of a small scene, rendered (simulation, or a look at a young scene)
        dict(name="lidar_render_small", op="lidar", n=4096, beams=32, azimuths=1024, channels=8, backward=False,
             ranges=False, moving=False),
        # one autograd step on a thumbnail camera: the smallest training call; ragged image
        dict(name="camera_step_small", op="camera", n=3000, width=157, height=93, channels=16, backward=True,
             moving=True, autograd=True),
        # one training view: a 1080p rolling-shutter camera over a road scene, forward and backward
        dict(name="camera_train_1080p", op="camera", n=500_000, width=1920, height=1080, channels=16, backward=True,
             moving=True, autograd=False),
        # one training sweep: a 128-beam lidar over two million Gaussians with measured ranges
        dict(name="lidar_train_sweep", op="lidar", n=2_000_000, beams=128, azimuths=2048, channels=8, backward=True,
             ranges=True, moving=True),
        # the training step of a camera and a lidar together, captured once and replayed
        dict(name="rig_train_step", op="rig", n=2_000_000, cameras=1, width=1920, height=1080, beams=128,
             azimuths=2048, backward=True),
        # one simulated frame of a vehicle's rig: six cameras and a lidar in one call per stage
        dict(name="rig_render_frame", op="rig", n=1_500_000, cameras=6, width=1280, height=720, beams=64,
             azimuths=1800, backward=False),
        # the lidar decoder in training: one sweep forward and backward
        dict(name="lidar_decode_sweep", op="lidar_decode", rays=262_144, channels=8, backward=True),
        # the lidar decoder over a batch of simulated sweeps
        dict(name="lidar_decode_batch", op="lidar_decode", rays=16_777_216, channels=8, backward=False),
        # the camera decoder on a rendered crop of odd size (simulation)
        dict(name="camera_decode_render", op="camera_decode", width=1237, height=713, features=16, embed=8,
             backward=False),
        # the camera decoder in training: a 1080p image forward and backward
        dict(name="camera_decode_train", op="camera_decode", width=1920, height=1080, features=16, embed=8,
             backward=True),
        # actors composed into the world frame and back, through autograd, once per training step
        dict(name="compose_train", op="compose", n=2_000_000, actors=64),
        # the regulariser and a relocation of dead Gaussians (a densification step)
        dict(name="densify", op="densify", n=2_000_000, dead=0.1, features=16),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["lidar", "camera", "rig", "lidar_decode", "camera_decode", "compose", "densify"])
    if op == "lidar":
        return dict(op=op, n=_log_int(rng, 2000, 2_000_000), beams=rng.choice([16, 32, 64, 128]),
                    azimuths=_log_int(rng, 250, 2048), channels=rng.choice([4, 8, 8, 13]),
                    backward=rng.random() < 0.6, ranges=rng.random() < 0.5, moving=rng.random() < 0.7)
    if op == "camera":
        w = _log_int(rng, 96, 1920)
        return dict(op=op, n=_log_int(rng, 2000, 500_000), width=w, height=max(40, int(w * rng.uniform(0.4, 0.56))),
                    channels=rng.choice([3, 8, 13, 16, 16]), backward=rng.random() < 0.6, moving=rng.random() < 0.7,
                    autograd=rng.random() < 0.4)
    if op == "rig":
        w = _log_int(rng, 160, 1280)
        return dict(op=op, n=_log_int(rng, 5000, 1_500_000), cameras=rng.randint(1, 4), width=w,
                    height=max(60, int(w * rng.uniform(0.45, 0.56))), beams=rng.choice([16, 32, 64]),
                    azimuths=_log_int(rng, 250, 1800), backward=rng.random() < 0.5)
    if op == "lidar_decode":
        return dict(op=op, rays=_log_int(rng, 3000, 16_000_000), channels=rng.choice([3, 8, 8, 16]),
                    backward=rng.random() < 0.6)
    if op == "camera_decode":
        w = _log_int(rng, 64, 1920)
        return dict(op=op, width=w, height=max(33, int(w * rng.uniform(0.4, 0.56))), features=rng.choice([7, 13, 16]),
                    embed=rng.choice([0, 8, 8]), backward=rng.random() < 0.6)
    if op == "compose":
        return dict(op=op, n=_log_int(rng, 3000, 2_000_000), actors=rng.choice([1, 7, 64, 300]))
    return dict(op="densify", n=_log_int(rng, 3000, 2_000_000), dead=round(rng.uniform(0.01, 0.4), 3),
                features=rng.choice([8, 13, 16]))


# ---- inputs: seeded draws on the GPU -------------------------------------------------------------
class _Draws:
    def __init__(self, seed):
        self.g = torch.Generator(device=DEV)
        self.g.manual_seed(int(seed))

    def normal(self, *shape):
        return torch.randn(*shape, generator=self.g, device=DEV)

    def uniform(self, *shape, lo=0.0, hi=1.0):
        return torch.rand(*shape, generator=self.g, device=DEV) * (hi - lo) + lo


def _gaussians(r, means, channels, moving):
    n = means.shape[0]
    ls = r.normal(n, 3) * 0.4 - 0.5
    q = r.normal(n, 4)
    q = q / q.norm(dim=1, keepdim=True)
    op = torch.sigmoid(r.normal(n))
    f = torch.cat([r.uniform(n, min(3, channels)), r.normal(n, max(0, channels - 3))], 1)
    vel = None
    if moving:   # a fifth of the scene moves
        vel = r.normal(n, 3) * 3.0 * (r.uniform(n, 1) < 0.2)
        vel = vel.contiguous()
    return B.GaussTensors(means.contiguous(), ls.contiguous(), q.contiguous(), op.contiguous(), vel, f.contiguous())


def _road(r, n):
    """A road slab ahead of a camera at its near end: most Gaussians hug the ground."""
    length = 40.0 * (n / 3000.0) ** 0.18
    x, y = r.uniform(n, lo=0.5, hi=length), r.uniform(n, lo=-15.0, hi=15.0)
    z = torch.where(r.uniform(n) < 0.7, (r.normal(n) * 0.1).abs(), r.uniform(n, hi=8.0))
    return torch.stack([x, y, z], 1)


def _field(r, n):
    """A flat box around the sensors: 40 m wide at 4096 Gaussians, 300 m at two million."""
    half = 20.0 * (n / 4096.0) ** 0.3255
    return torch.stack([r.uniform(n, lo=-half, hi=half), r.uniform(n, lo=-half, hi=half),
                        r.uniform(n, lo=-3.0, hi=3.0)], 1)


def _yaw(deg):
    c, s = math.cos(math.radians(deg)), math.sin(math.radians(deg))
    return np.array([[c, -s, 0.0], [s, c, 0.0], [0.0, 0.0, 1.0]])


def _camera(width, height, channels, yaw=0.0, pos=(0.0, 0.0, 1.5), ego=(15.0, 0.0, 0.0)):
    axes = np.array([[0.0, 0.0, 1.0], [-1.0, 0.0, 0.0], [0.0, -1.0, 0.0]])
    R = (_yaw(yaw) @ axes).T
    f32 = lambda a: np.asarray(a, np.float32)
    fx = float(np.float32(0.78 * width))
    return SimpleNamespace(R=f32(R), t=f32(-R @ np.asarray(pos)), fx=fx, fy=fx, cx=width / 2.0, cy=height / 2.0,
                           width=width, height=height, lin_vel=f32(R @ np.asarray(ego)), ang_vel=f32(np.zeros(3)),
                           t_rs=float(np.float32(0.03)), eps2d=float(np.float32(0.3)), near=float(np.float32(0.2)),
                           far=1.0e4, jac_clamp=float(np.float32(1.3)), feat_offset=0, n_channels=channels, tile_w=16,
                           tile_h=16, time_offset=0.0, n_rays=width * height)


def _lidar(beams, azimuths, channels, offset, ranges=None, ego=(15.0, 0.0, 0.0), sweep=0.1):
    w = np.linspace(-25.0, 15.0, 20001)      # channels are denser near the horizon
    dens = 1.0 + 3.0 * np.exp(-(w / 4.0) ** 2)
    cdf = np.concatenate([[0.0], np.cumsum(0.5 * (dens[1:] + dens[:-1]) * np.diff(w))])
    ch = np.radians(np.interp((np.arange(beams) + 0.5) / beams, cdf / cdf[-1], w))
    per = 8
    m = beams // per
    inner = [0.5 * (ch[k * per - 1] + ch[k * per]) for k in range(1, m)]
    bounds = np.array([ch[0] - 0.5 * (ch[1] - ch[0]), *inner, ch[-1] + 0.5 * (ch[-1] - ch[-2])])
    res = 2.0 * math.pi / azimuths
    j = np.arange(azimuths)
    f32 = lambda a: np.asarray(a, np.float32)
    return SimpleNamespace(R=f32(np.eye(3)), t=f32(np.zeros(3)), lin_vel=f32(ego), ang_vel=f32(np.zeros(3)),
                           t_rs=float(np.float32(sweep)), eps2d=float(np.float32(res * (ch[-1] - ch[0]) / (beams - 1))),
                           r_min=0.5, r_max=250.0, az_res=float(np.float32(res)), tile_az=32,
                           n_az_tiles=-(-azimuths // 32), n_el_tiles=m, elev_bounds=f32(bounds),
                           ray_az=f32(np.tile((j + 0.5) * res, beams)), ray_el=f32(np.repeat(ch, azimuths)),
                           ray_t=f32(np.tile(((j + 0.5) / azimuths - 0.5) * sweep, beams)), ray_range=ranges,
                           los_eps=float(np.float32(0.8)), feat_offset=offset, n_channels=channels,
                           n_rays=beams * azimuths)


def _ranges(r, rays):
    return torch.exp(r.uniform(rays, lo=math.log(2.0), hi=math.log(100.0))).cpu().numpy()


def _flat(tensors):
    """Accumulators shaped like `tensors` as views of one buffer (16-byte aligned), cleared at once."""
    ends = np.cumsum([0] + [(t.numel() + 3) // 4 * 4 for t in tensors])
    buf = torch.zeros(int(ends[-1]), device=DEV)
    return buf, [buf[int(a):int(a) + t.numel()].view(t.shape) for a, t in zip(ends, tensors)]


def _upstream(r, floats, rays):
    return r.normal(max(1, floats)), 0.01 * r.normal(max(1, rays)), r.normal(max(1, rays))


def _scene(case, seed):
    """(Gaussians, cameras, lidars, the draws for what follows) of a render case."""
    r = _Draws(seed)
    op = case["op"]
    if op == "camera":
        g = _gaussians(r, _road(r, case["n"]), case["channels"], case["moving"])
        return g, [_camera(case["width"], case["height"], case["channels"])], [], r
    if op == "lidar":
        g = _gaussians(r, _field(r, case["n"]), case["channels"] + 3, case["moving"])
        rng = _ranges(r, case["beams"] * case["azimuths"]) if case["ranges"] else None
        return g, [], [_lidar(case["beams"], case["azimuths"], case["channels"], 3, rng)], r
    g = _gaussians(r, _field(r, case["n"]), 16, True)
    yaws = [0.0, 180.0, 60.0, -60.0, 120.0, -120.0]
    cams = [_camera(case["width"], case["height"], 16, yaws[k], (0.0, 0.0, 0.0)) for k in range(case["cameras"])]
    rng = _ranges(r, case["beams"] * case["azimuths"]) if case["backward"] else None
    return g, cams, [_lidar(case["beams"], case["azimuths"], 8, 3, rng)], r


# ---- prepare -------------------------------------------------------------------------------------
def prepare(case, seed):
    return _PREPARE[case["op"]](case, seed)


def _prepare_render(case, seed):
    g, cams, lids, r = _scene(case, seed)
    rig = B.Rig(cams, lids, DEV)
    s = SimpleNamespace(op=case["op"], case=case, g=g, rig=rig, pipe=None, grads=None)
    s.sp = B.SensorPass(rig, 0, len(cams) + len(lids), g.n, 1, DEV, batched=case["op"] == "rig")
    s.sp.fit_capacity(g)
    if case["backward"]:
        s.dF, s.dD, s.dA = _upstream(r, s.sp.n_feat, s.sp.n_rays)
        s.dL = 0.1 * r.normal(s.sp.n_rays) if lids else None
        if s.dL is not None and cams:
            s.dL[:int(s.sp.ray_off[len(cams)])] = 0.0
        have = [t for t in (g.means, g.log_scales, g.quats, g.opacities, g.velocities, g.features) if t is not None]
        s.grad_buffer, views = _flat(have)
        s.grads = B.GaussTensors(*views[:4], views[4] if g.velocities is not None else None, views[-1])
        if case["op"] == "rig":
            s.pipe = B.Pipeline(s.sp, g, grads=s.grads, dF=s.dF, dD=s.dD, dA=s.dA, d_los=s.dL)
        if case.get("autograd"):
            s.leaves = [t if t is None else t.requires_grad_(True)
                        for t in (g.means, g.log_scales, g.quats, g.opacities, g.velocities, g.features)]
    s.lidar_rays = slice(int(s.sp.ray_off[len(cams)]), s.sp.n_rays) if lids else None
    return s


def _mlp(r, channels):
    w1 = r.normal(32, channels + 3) * math.sqrt(2.0 / (channels + 3))
    return B.LidarMLP(w1.contiguous(), 0.1 * r.normal(32), r.normal(2, 32) * math.sqrt(1.0 / 32), 0.1 * r.normal(2))


def _decode_inputs(case, seed):
    r = _Draws(seed)
    n, c = case["rays"], case["channels"]
    return r, r.normal(n, c), r.uniform(n, hi=6.283), r.uniform(n, lo=-0.44, hi=0.26), _mlp(r, c)


def _prepare_lidar_decode(case, seed):
    r, feat, az, el, mlp = _decode_inputs(case, seed)
    s = SimpleNamespace(op="lidar_decode", case=case, feat=feat, az=az, el=el, mlp=mlp)
    if case["backward"]:
        n = case["rays"]
        s.dI, s.dP = r.normal(n), r.normal(n)
        s.grad_buffer, (s.d_feat, *w) = _flat([feat] + [getattr(mlp, f) for f in B.MLP_FIELDS])
        s.d_mlp = dict(zip(B.MLP_FIELDS, w))
        need = int(B.load().splat_lidar_decode_workspace_bytes(n, case["channels"]))
        s.ws = torch.empty(max(need, 1), dtype=torch.uint8, device=DEV)
    return s


def _cnn_inputs(case, seed):
    r = _Draws(seed)
    cin = case["features"] + 3 + case["embed"]
    he = lambda co, ci: r.normal(co, ci, 3, 3) * math.sqrt(2.0 / (9 * ci))
    cnn = B.CameraCNN(0.3 * r.normal(case["embed"]), he(32, cin), 0.05 * r.normal(32), [he(32, 32) for _ in range(4)],
                      [0.05 * r.normal(32) for _ in range(4)], r.normal(6, 32) * math.sqrt(1.0 / 32), 0.05 * r.normal(6))
    cam = _camera(case["width"], case["height"], case["features"], 25.0)
    n = cam.n_rays
    feat = torch.cat([r.uniform(n, 3), r.normal(n, case["features"] - 3)], 1).contiguous()
    return r, cam, cnn, feat


def _prepare_camera_decode(case, seed):
    r, cam, cnn, feat = _cnn_inputs(case, seed)
    s = SimpleNamespace(op="camera_decode", case=case, cam=cam, cnn=cnn, feat=feat,
                        ws=B.camera_decode_workspace(cam, DEV))
    if case["backward"]:
        s.d_image = r.normal(cam.n_rays * 3)
        s.grad_buffer, v = _flat([feat, cnn.embed, cnn.w_in, cnn.b_in, cnn.w_out, cnn.b_out, *cnn.w_block,
                                  *cnn.b_block])
        s.d_feat = v[0]
        s.d_cnn = dict(embed=v[1], w_in=v[2], b_in=v[3], w_out=v[4], b_out=v[5], w_block=v[6:10], b_block=v[10:14])
    return s


def _compose_inputs(case, seed):
    r = _Draws(seed)
    n, A = case["n"], case["actors"]
    n_act = int(round(0.3 * n))
    road = _road(r, n - n_act)
    local = r.uniform(n_act, 3, lo=-1.0) * torch.tensor([2.25, 1.0, 0.8], device=DEV)
    aid = torch.randint(0, A, (n_act,), generator=r.g, device=DEV).sort().values
    g = _gaussians(r, torch.cat([road, local]), 3, True)
    g.velocities[n - n_act:] = 0.0
    actor_id = torch.cat([torch.full((n - n_act,), -1, device=DEV), aid]).to(torch.int32)
    yaw = r.uniform(A, lo=-math.pi, hi=math.pi)
    z = torch.zeros(A, device=DEV)
    rot = torch.stack([torch.cos(yaw / 2), 0.01 * r.normal(A), 0.01 * r.normal(A), torch.sin(yaw / 2)], 1)
    rot = (rot / rot.norm(dim=1, keepdim=True)).contiguous()
    trans = torch.stack([r.uniform(A, lo=5.0, hi=100.0), r.uniform(A, lo=-12.0, hi=12.0), z + 0.8], 1).contiguous()
    rot_off = torch.cat([torch.ones(A, 1, device=DEV), 0.01 * r.normal(A, 3)], 1).contiguous()
    lin = torch.stack([10.0 + 3.0 * r.normal(A), z, z], 1).contiguous()
    ang = torch.stack([z, z, 0.2 * r.normal(A)], 1).contiguous()
    const = [actor_id, rot, trans, lin]
    leaves = [g.means, g.quats, g.velocities, rot_off, 0.05 * r.normal(A, 3), 0.1 * r.normal(A, 3), ang]
    ups = [r.normal(n, 3), r.normal(n, 4), r.normal(n, 3)]
    return const, leaves, ups


def _prepare_compose(case, seed):
    const, leaves, ups = _compose_inputs(case, seed)
    return SimpleNamespace(op="compose", case=case, const=const, leaves=[t.requires_grad_(True) for t in leaves],
                           ups=ups)


def _densify_inputs(case, seed):
    r = _Draws(seed)
    n = case["n"]
    g = _gaussians(r, _field(r, n), case["features"], True)
    dead = r.uniform(n) < case["dead"]
    g.opacities = torch.where(dead, r.uniform(n, lo=1e-4, hi=0.0049), g.opacities.clamp(min=0.006)).contiguous()
    u = torch.randint(-2 ** 31, 2 ** 31, (n,), generator=r.g, device=DEV, dtype=torch.int64).to(torch.int32)
    return g, u


def _prepare_densify(case, seed):
    g, u = _densify_inputs(case, seed)
    need = int(B.load().splat_mcmc_relocate_workspace_bytes(case["n"]))
    return SimpleNamespace(op="densify", case=case, g=g, u=u, opacities=g.opacities.clone(),
                           log_scales=g.log_scales.clone(), value=torch.zeros(1, device=DEV),
                           grads=B.zeros_like_grads(g), ws=torch.empty(need, dtype=torch.uint8, device=DEV))


_PREPARE = dict(camera=_prepare_render, lidar=_prepare_render, rig=_prepare_render, lidar_decode=_prepare_lidar_decode,
                camera_decode=_prepare_camera_decode, compose=_prepare_compose, densify=_prepare_densify)


# ---- run -----------------------------------------------------------------------------------------
def run(state):
    return _RUN[state.op](state)


def _grad_outputs(g):
    return dict(means=g.means, log_scales=g.log_scales, quats=g.quats, opacities=g.opacities, velocities=g.velocities,
                features=g.features)


def _run_render(s):
    if s.case.get("autograd") and s.case["backward"]:
        F, D, A = B.SplatRenderFn.apply(s.sp, B.BOX, *s.leaves)
        grads = torch.autograd.grad([F, D, A], [t for t in s.leaves if t is not None], [s.dF, s.dD, s.dA])
        return dict(feat=F, depth=D, alpha=A, grads=list(grads))
    if s.pipe is not None:
        s.pipe.run()
        o = s.sp.outputs()
    else:
        o = s.sp.render(s.g)
        if s.grads is not None:
            s.grad_buffer.zero_()
            s.sp.raster_bwd(s.g, s.dF, s.dD, s.dA, s.grads, d_los=s.dL)
    out = dict(feat=o["feat"], depth=o["depth"], alpha=o["alpha"], t_final=o["t_final"], last=o["last"])
    if s.lidar_rays is not None:    # cameras have neither a median range nor a line-of-sight sum
        out.update(median=o["median"][s.lidar_rays], los=o["los"][s.lidar_rays])
    if s.grads is not None:
        out["grads"] = _grad_outputs(s.grads)
    return out


def _run_lidar_decode(s):
    I, P = B.lidar_decode(s.feat, s.az, s.el, s.mlp)
    if not s.case["backward"]:
        return dict(intensity=I, drop=P)
    s.grad_buffer.zero_()
    B.lidar_decode_bwd(s.feat, s.az, s.el, s.mlp, s.dI, s.dP, s.d_feat, s.d_mlp, s.ws)
    return dict(intensity=I, drop=P, d_feat=s.d_feat, **s.d_mlp)


def _run_camera_decode(s):
    image = B.camera_decode(s.cam, s.feat, s.cnn, s.ws)
    if not s.case["backward"]:
        return dict(image=image)
    s.grad_buffer.zero_()
    B.camera_decode_bwd(s.cam, s.feat, s.cnn, s.d_image, s.d_feat, s.d_cnn, s.ws)
    return dict(image=image, d_feat=s.d_feat, **s.d_cnn)


def _run_compose(s):
    w = B.ComposeFn.apply(*s.const, *s.leaves)
    return dict(world=list(w), grads=list(torch.autograd.grad(w, s.leaves, s.ups)))


def _run_densify(s):
    # what the optimiser's step left: opacities and scales of this iteration
    s.g.opacities.copy_(s.opacities)
    s.g.log_scales.copy_(s.log_scales)
    s.value.zero_()
    s.grads.opacities.zero_()
    s.grads.log_scales.zero_()
    B.mcmc_regularizer(s.g, s.value, s.grads)
    target, moved = B.mcmc_relocate(s.g, s.u, ws=s.ws)
    return dict(value=s.value, d_opacities=s.grads.opacities, d_log_scales=s.grads.log_scales, target=target,
                moved=moved, state=_grad_outputs(s.g))


_RUN = dict(camera=_run_render, lidar=_run_render, rig=_run_render, lidar_decode=_run_lidar_decode,
            camera_decode=_run_camera_decode, compose=_run_compose, densify=_run_densify)


# ---- work ----------------------------------------------------------------------------------------
def work(case):
    op = case["op"]
    if op in ("camera", "lidar", "rig"):
        n = case["n"]
        sensors = []     # (rays, channels, bytes of a ray's inputs, of its outputs beside the features)
        if op != "lidar":
            k = case.get("cameras", 1)
            sensors.append((k * case["width"] * case["height"], case.get("channels", 16), 0, 16))
        if op != "camera":
            sensors.append((case["beams"] * case["azimuths"], case["channels"] if op == "lidar" else 8, 12, 24))
        ctot = {"camera": case.get("channels", 0), "lidar": case.get("channels", 0) + 3, "rig": 16}[op]
        row = 4 * (3 + 3 + 4 + 1 + (3 if case.get("moving", True) else 0) + ctot)
        views = case.get("cameras", 1) + (1 if op == "rig" else 0)
        b = n * row + sum(r * (4 * c + i + o) for r, c, i, o in sensors)
        f = n * views * 250.0 + sum(r * PAIRS_PER_RAY * (22.0 + 2 * c) for r, c, _, _ in sensors)
        if case["backward"]:
            b += n * row + sum(r * 4 * (c + 2) for r, c, _, _ in sensors)
            f += n * views * 250.0 + sum(r * PAIRS_PER_RAY * 2 * (22.0 + 2 * c) for r, c, _, _ in sensors)
        return dict(bytes=b, flops=f)
    if op == "lidar_decode":
        n, c = case["rays"], case["channels"]
        f = n * 2.0 * (32 * (c + 3) + 64)
        return dict(bytes=n * 4 * (c + 4 + ((c + 2) if case["backward"] else 0)), flops=f * (3 if case["backward"] else 1))
    if op == "camera_decode":
        n, c = case["width"] * case["height"], case["features"]
        f = n * 2.0 * (9 * 32 * (c + 3 + case["embed"]) + 4 * 9 * 32 * 32 + 6 * 32)
        return dict(bytes=n * 4 * (c + 3 + ((c + 3) if case["backward"] else 0)), flops=f * (3 if case["backward"] else 1))
    n = case["n"]
    if op == "compose":
        return dict(bytes=n * 4.0 * (11 + 10 + 10 + 10), flops=n * 250.0)
    row = 4 * (3 + 3 + 4 + 1 + 3 + case["features"])
    return dict(bytes=n * 4.0 * (4 + 4 + 4 + 4 + 1 + 1) + 2.0 * case["dead"] * n * row, flops=n * 30.0)


# ---- exact: plain torch in 64 bits ----------------------------------------------------------------
def exact(case, seed):
    return _EXACT[case["op"]](case, seed)


def _rotation(q):
    w, x, y, z = (q / q.norm(dim=-1, keepdim=True)).unbind(-1)
    return torch.stack([1 - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y),
                        2 * (x * y + w * z), 1 - 2 * (x * x + z * z), 2 * (y * z - w * x),
                        2 * (x * z - w * y), 2 * (y * z + w * x), 1 - 2 * (x * x + y * y)], -1).reshape(-1, 3, 3)


def _rows(*rows):
    return torch.stack([torch.stack(r, -1) for r in rows], -2)


def _project64(p, sen, lidar):
    """Means, velocities, conics, opacities, depths and range velocities of one sensor, with the
    boxes and the culling (decisions, not differentiated)."""
    t64 = lambda a: torch.as_tensor(np.asarray(a, np.float64), device=DEV)
    means, ls, q, op, vel = p
    R = t64(sen.R)
    M = R @ (_rotation(q) * torch.exp(ls)[:, None, :])
    mu = means @ R.T + t64(sen.t)
    rel = -torch.linalg.cross(t64(sen.ang_vel).expand_as(mu), mu, dim=-1) - t64(sen.lin_vel)
    if vel is not None:
        rel = rel + vel @ R.T
    x, y, z = mu.unbind(-1)
    zero = torch.zeros_like(x)
    if lidar:
        r = mu.norm(dim=-1)
        rho = torch.sqrt(x * x + y * y)
        ok = (r >= sen.r_min) & (r <= sen.r_max) & (rho >= 1e-4 * r)
        x, y, z, r, rho = (torch.where(ok, a, torch.ones_like(a)) for a in (x, y, z, r, rho))
        phi = torch.atan2(y, x)
        phi = torch.where(phi < 0, phi + 2 * math.pi, phi)
        mean = torch.stack([phi, torch.asin((z / r).clamp(-1, 1))], -1)
        J = _rows((-y / rho ** 2, x / rho ** 2, zero), (-x * z / (r * r * rho), -y * z / (r * r * rho), rho / (r * r)))
        vr = (x * rel[:, 0] + y * rel[:, 1] + z * rel[:, 2]) / r
        depth = r
    else:
        ok = (z > sen.near) & (z < sen.far)
        z = torch.where(ok, z, torch.ones_like(z))
        tx, ty = x / z, y / z
        mean = torch.stack([sen.fx * tx + sen.cx, sen.fy * ty + sen.cy], -1)
        lx, ly = sen.jac_clamp * 0.5 * sen.width / sen.fx, sen.jac_clamp * 0.5 * sen.height / sen.fy
        tx, ty = tx.clamp(-lx, lx), ty.clamp(-ly, ly)
        J = _rows((sen.fx / z, zero, -sen.fx * tx / z), (zero, sen.fy / z, -sen.fy * ty / z))
        vr, depth = zero, z
    T = J @ M
    S = T @ T.transpose(1, 2)
    v2 = (J @ rel[..., None])[..., 0]
    a, b, c = S[:, 0, 0] + sen.eps2d, S[:, 0, 1], S[:, 1, 1] + sen.eps2d
    det = a * c - b * b
    det0 = (torch.linalg.cross(T[:, 0], T[:, 1], dim=-1) ** 2).sum(-1)
    conic = torch.stack([c / det, -b / det, a / det], -1)
    o = op * torch.sqrt((det0 / det).clamp(min=1e-300))
    with torch.no_grad():
        ext = 3 * torch.sqrt(torch.stack([a, c], -1)) + v2.abs() * (0.5 * sen.t_rs)
        lo, hi = mean - ext, mean + ext
        ok = ok & (o >= 1.0 / 255.0)
        if lidar:
            ok &= (hi[:, 1] > float(sen.elev_bounds[0])) & (lo[:, 1] < float(sen.elev_bounds[-1]))
        else:
            ok &= (lo[:, 0] < sen.width) & (hi[:, 0] > 0) & (lo[:, 1] < sen.height) & (hi[:, 1] > 0)
        idx = torch.nonzero(ok)[:, 0]
        idx = idx[torch.sort(depth[idx], stable=True).indices]
    return (mean, v2, conic, o, depth, vr), lo[idx], hi[idx], idx


def _composite64(q, lo, hi, feat, pts, t, thr, lidar):
    """Front-to-back blending of the sorted Gaussians at a chunk of rays."""
    mean, v2, conic, o, depth, vr = q
    d = pts[:, None, :] - (mean[None] + v2[None] * t[:, None, None])
    dx, dy = d[..., 0], d[..., 1]
    if lidar:
        dx = torch.remainder(dx + math.pi, 2 * math.pi) - math.pi
        inside = torch.remainder(pts[:, None, 0] - lo[None, :, 0], 2 * math.pi) < (hi - lo)[None, :, 0]
    else:
        inside = (pts[:, None, 0] >= lo[None, :, 0]) & (pts[:, None, 0] < hi[None, :, 0])
    inside = inside & (pts[:, None, 1] >= lo[None, :, 1]) & (pts[:, None, 1] < hi[None, :, 1])
    power = 0.5 * (conic[:, 0] * dx * dx + conic[:, 2] * dy * dy) + conic[:, 1] * dx * dy
    alpha = (o * torch.exp(-power)).clamp(max=0.99)
    with torch.no_grad():
        keep = inside & (alpha >= 1.0 / 255.0)
        keep &= torch.cumprod(1 - torch.where(keep, alpha, torch.zeros_like(alpha)), 1) >= 1e-4
    a = torch.where(keep, alpha, torch.zeros_like(alpha))
    after = torch.cumprod(1 - a, 1)
    before = torch.cat([torch.ones_like(after[:, :1]), after[:, :-1]], 1)
    w = a * before
    rng = depth[None] + vr[None] * t[:, None] if lidar else depth[None].expand_as(w)
    out = [w @ feat, (w * rng).sum(1), 1 - after[:, -1], after[:, -1]]
    if lidar:
        with torch.no_grad():
            first = keep & (after < 0.5) & (before >= 0.5)
            med = (first * rng).sum(1)
        los = (a * (keep & (rng.detach() < thr[:, None]))).sum(1) if thr is not None else torch.zeros_like(t)
        out += [med, los]
    return out


def _exact_render(case, seed):
    rays = 0 if case["op"] == "lidar" else case.get("cameras", 1) * case["width"] * case["height"]
    rays += 0 if case["op"] == "camera" else case["beams"] * case["azimuths"]
    if float(rays) * case["n"] > EXACT_PAIRS:
        return None
    g, cams, lids, r = _scene(case, seed)
    back = case["backward"]
    leaves = [None if t is None else t.detach().to(F64).requires_grad_(back)
              for t in (g.means, g.log_scales, g.quats, g.opacities, g.velocities, g.features)]
    if back:
        floats = sum(s.n_rays * s.n_channels for s in cams + lids)
        dF, dD, dA = (x.to(F64) for x in _upstream(r, floats, rays))
        dL = 0.1 * r.normal(rays).to(F64) if lids else None
    parts, f0, r0 = [], 0, 0
    for sen in cams + lids:
        lidar = sen in lids
        q, lo, hi, idx = _project64(leaves[:5], sen, lidar)
        feat = leaves[5][:, sen.feat_offset:sen.feat_offset + sen.n_channels]
        src = [x[idx] for x in q] + [feat[idx]]
        cut = [x.detach().requires_grad_(back) for x in src]
        if lidar:
            pts = torch.stack([torch.as_tensor(sen.ray_az, device=DEV), torch.as_tensor(sen.ray_el, device=DEV)], 1).to(F64)
            t = torch.as_tensor(sen.ray_t, device=DEV).to(F64)
        else:
            i = torch.arange(sen.n_rays, device=DEV)
            row = (i // sen.width).to(F64) + 0.5
            pts = torch.stack([(i % sen.width).to(F64) + 0.5, row], 1)
            t = (row / sen.height - 0.5) * sen.t_rs
        has = lidar and sen.ray_range is not None
        thr = torch.as_tensor(sen.ray_range, device=DEV).to(F64) - sen.los_eps if has else None
        step = max(1, int(2.0e7 / max(1, idx.numel())))
        got = []
        for k in range(0, sen.n_rays, step):
            e = min(sen.n_rays, k + step)
            if idx.numel() == 0:
                z = torch.zeros(e - k, dtype=F64, device=DEV)
                got.append([torch.zeros(e - k, sen.n_channels, dtype=F64, device=DEV), z, z, z + 1, z, z][:6 if lidar else 4])
                continue
            out = _composite64(cut[:6], lo, hi, cut[6], pts[k:e], t[k:e], None if thr is None else thr[k:e], lidar)
            if back:
                C = sen.n_channels
                up = (out[0] * dF[f0 + k * C:f0 + e * C].reshape(-1, C)).sum() + (out[1] * dD[r0 + k:r0 + e]).sum() \
                    + (out[2] * dA[r0 + k:r0 + e]).sum()
                if has:
                    up = up + (out[5] * dL[r0 + k:r0 + e]).sum()
                up.backward()
            got.append([x.detach() for x in out])
        if back and idx.numel():
            pairs = [(x, y.grad) for x, y in zip(src, cut) if y.grad is not None and x.requires_grad]
            torch.autograd.backward([x for x, _ in pairs], [y for _, y in pairs])
        parts.append([torch.cat([x[j] for x in got]) for j in range(len(got[0]))])
        f0, r0 = f0 + sen.n_rays * sen.n_channels, r0 + sen.n_rays
    cat = lambda j: torch.cat([p[j].reshape(-1) for p in parts])
    grad = lambda t: None if t is None else torch.zeros_like(t) if t.grad is None else t.grad
    if case.get("autograd") and back:
        return dict(feat=cat(0), depth=cat(1), alpha=cat(2), grads=[grad(t) for t in leaves if t is not None])
    out = dict(feat=cat(0), depth=cat(1), alpha=cat(2), t_final=cat(3), last=None)
    if lids:
        out.update(median=parts[-1][4], los=parts[-1][5])
    if back:
        names = ("means", "log_scales", "quats", "opacities", "velocities", "features")
        out["grads"] = {k: grad(t) for k, t in zip(names, leaves)}
    return out


def _exact_lidar_decode(case, seed):
    r, feat, az, el, mlp = _decode_inputs(case, seed)
    back = case["backward"]
    w = [getattr(mlp, f).to(F64).requires_grad_(back) for f in B.MLP_FIELDS]
    n = case["rays"]
    dI, dP = (r.normal(n), r.normal(n)) if back else (None, None)
    I, P, dF = [], [], []
    for k in range(0, n, 1 << 21):
        e = min(n, k + (1 << 21))
        x = feat[k:e].to(F64).requires_grad_(back)
        a, b = az[k:e].to(F64), el[k:e].to(F64)
        d = torch.stack([torch.cos(b) * torch.cos(a), torch.cos(b) * torch.sin(a), torch.sin(b)], 1)
        h = torch.relu(torch.cat([x, d], 1) @ w[0].T + w[1])
        y = torch.sigmoid(h @ w[2].T + w[3])
        if back:
            torch.autograd.backward([y], [torch.stack([dI[k:e], dP[k:e]], 1).to(F64)])
            dF.append(x.grad)
        I.append(y[:, 0].detach())
        P.append(y[:, 1].detach())
    out = dict(intensity=torch.cat(I), drop=torch.cat(P))
    if back:
        out.update(d_feat=torch.cat(dF), **{f: t.grad for f, t in zip(B.MLP_FIELDS, w)})
    return out


def _exact_camera_decode(case, seed):
    r, cam, cnn, feat = _cnn_inputs(case, seed)
    back = case["backward"]
    H, W = cam.height, cam.width
    leaf = lambda t: t.to(F64).requires_grad_(back)
    x = leaf(feat)
    emb, w_in, b_in, w_out, b_out = (leaf(t) for t in (cnn.embed, cnn.w_in, cnn.b_in, cnn.w_out, cnn.b_out))
    wb, bb = [leaf(t) for t in cnn.w_block], [leaf(t) for t in cnn.b_block]
    R = torch.as_tensor(np.asarray(cam.R, np.float64), device=DEV)
    i = torch.arange(H * W, device=DEV)
    d = torch.stack([((i % W).to(F64) + 0.5 - cam.cx) / cam.fx, ((i // W).to(F64) + 0.5 - cam.cy) / cam.fy,
                     torch.ones(H * W, dtype=F64, device=DEV)], 1)
    d = (d / d.norm(dim=1, keepdim=True)) @ R

    def conv(h, w, b):
        c = h.shape[1]
        p = torch.nn.functional.pad(h.reshape(H, W, c), (0, 0, 1, 1, 1, 1))
        y = b.expand(H * W, -1)
        for ky in range(3):
            for kx in range(3):
                y = y + p[ky:ky + H, kx:kx + W].reshape(H * W, c) @ w[:, :, ky, kx].T
        return y

    h = torch.relu(conv(torch.cat([x, d, emb.expand(H * W, -1)], 1), w_in, b_in))
    for k in range(2):
        h = torch.relu(h + conv(torch.relu(conv(h, wb[2 * k], bb[2 * k])), wb[2 * k + 1], bb[2 * k + 1]))
    z = h @ w_out.T + b_out
    image = (z[:, :3] * x[:, :3] + z[:, 3:]).reshape(-1)
    if not back:
        return dict(image=image)
    image.backward(r.normal(H * W * 3).to(F64))
    grad = lambda t: torch.zeros_like(t) if t.grad is None else t.grad
    return dict(image=image.detach(), d_feat=x.grad, embed=grad(emb), w_in=w_in.grad, b_in=b_in.grad,
                w_block=[t.grad for t in wb], b_block=[t.grad for t in bb], w_out=w_out.grad, b_out=b_out.grad)


def _product(a, b):
    w, x, y, z = a.unbind(-1)
    s, i, j, k = b.unbind(-1)
    return torch.stack([w * s - x * i - y * j - z * k, w * i + x * s + y * k - z * j, w * j - x * k + y * s + z * i,
                        w * k + x * j - y * i + z * s], -1)


def _exact_compose(case, seed):
    (aid, rot, trans, lin), leaves, ups = _compose_inputs(case, seed)
    leaves = [t.to(F64).requires_grad_(True) for t in leaves]
    m, q, v, dq, dt, dv, w = leaves
    rot, trans, lin = rot.to(F64), trans.to(F64), lin.to(F64)
    qa = _product(rot / rot.norm(dim=1, keepdim=True), dq / dq.norm(dim=1, keepdim=True))
    R, ta, va = _rotation(qa), trans + dt, lin + dv
    moving = (aid >= 0)[:, None]
    k = aid.clamp(min=0).to(torch.int64)
    mw = torch.where(moving, (R[k] @ m[..., None])[..., 0] + ta[k], m)
    qw = torch.where(moving, _product(qa[k], q), q)
    vw = torch.where(moving, (R[k] @ (torch.linalg.cross(w[k], m, dim=-1) + va[k])[..., None])[..., 0], v)
    grads = torch.autograd.grad([mw, qw, vw], leaves, [u.to(F64) for u in ups])
    return dict(world=[mw.detach(), qw.detach(), vw.detach()], grads=list(grads))


def _exact_densify(case, seed):
    g, u = _densify_inputs(case, seed)
    o, ls = g.opacities.to(F64), g.log_scales.to(F64)
    value = (B.MCMC_LAMBDA_O * o.abs().sum() + B.MCMC_LAMBDA_S * torch.exp(ls).sum()).reshape(1)
    dead = g.opacities <= B.MCMC_DEAD_OPACITY
    wt = torch.where(dead, torch.zeros_like(o), torch.floor(o.clamp(max=1) * 2.0 ** 24)).to(torch.int64)
    cum = torch.cumsum(wt, 0)
    total = int(cum[-1])
    draw64 = u.to(torch.int64) & 0xFFFFFFFF      # floor(draw * total / 2^32) in 64-bit pieces
    A, L = draw64 * (total >> 24), draw64 * (total & 0xFFFFFF)
    pick = (A >> 8) + ((((A & 0xFF) << 24) + L) >> 32)
    tgt = torch.searchsorted(cum, pick, right=True).clamp(max=case["n"] - 1)
    rows = torch.nonzero(dead)[:, 0]
    src = tgt[rows]
    N = (1 + torch.bincount(src, minlength=case["n"])).clamp(max=B.MCMC_N_MAX)
    on = -torch.expm1(torch.log1p(-o) / N)
    total_k = torch.zeros_like(o)
    binom = torch.ones_like(o)
    for k in range(1, int(N.max()) + 1):
        binom = binom * (N - k + 1).clamp(min=0) / k
        total_k += binom * (-1.0) ** (k + 1) * on ** k / math.sqrt(k)
    hit = N > 1
    o2 = torch.where(hit, on, o)
    ls2 = torch.where(hit[:, None], ls + torch.log(o / total_k)[:, None], ls)
    arrays = dict(means=g.means.to(F64), log_scales=ls2, quats=g.quats.to(F64), opacities=o2,
                  velocities=g.velocities.to(F64), features=g.features.to(F64))
    for k in arrays:
        arrays[k] = arrays[k].clone()
        arrays[k][rows] = arrays[k][src]
    return dict(value=value, d_opacities=B.MCMC_LAMBDA_O * torch.sign(o), d_log_scales=B.MCMC_LAMBDA_S * torch.exp(ls),
                target=None, moved=None, state=arrays)


_EXACT = dict(camera=_exact_render, lidar=_exact_render, rig=_exact_render, lidar_decode=_exact_lidar_decode,
              camera_decode=_exact_camera_decode, compose=_exact_compose, densify=_exact_densify)
