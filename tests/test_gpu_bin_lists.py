"""Binning alone, whole: entry numbers and every tile's list, bit for bit against the same integers
computed in numpy from the projected records (rectangles, depths), at record counts around the wavefront
(64), the write line (8 and 16 records), the scans' blocks (2048 pairs, 4096 counts) and the emission's
chunks, on both sides of the sort in one workgroup (8192 records), with few and with many supertiles per
record, with equal depths, for one camera, one lidar (rectangles across the azimuth seam), both in one
call, and with a camera of exactly 256 and of more than 256 tile columns (rectangles packed in 32 bits,
and not)."""
import numpy as np
import pytest
import torch

from scenes import synthetic as S
from tests.gpu_helpers import tile_lists_gpu

pytestmark = pytest.mark.gpu


def _binding():
    from paper_2411_16816_amd import binding
    binding.load()
    return binding


def _scene(n, size, which):
    rng = np.random.default_rng(n + int(100 * size))
    g = S.random_gaussians(rng, rng.uniform([-30, -30, -3], [30, 30, 3], (n, 3)), 11, moving_frac=0.3)
    g.log_scales += np.float32(np.log(size))
    size_px = {"w": (4110, 60), "e": (4096, 60)}.get(which[0], (700, 300))
    cam = S.make_camera(np.zeros(3), 10.0, *size_px, 320.0, n_channels=8) if which[0] != "l" else None
    lid = S.make_lidar(np.zeros(3), 0.0, 32, -25.0, 15.0, 900, feat_offset=8, n_channels=3) if which[-1] == "l" else None
    return g, [cam] if cam else [], [lid] if lid else []


def _sort_key(dkey):
    bits = dkey.astype(np.uint64)
    e = (bits >> np.uint64(52)).astype(np.int64) - (1023 - 16)
    key = (np.clip(e, 0, 31) << 27) | ((bits & np.uint64(0xFFFFFFFFFFFFF)) >> np.uint64(25)).astype(np.int64)
    return np.where(e < 0, 0, np.where(e > 31, 0xFFFFFFFF, key))


def _expected(rig, sp, n):
    nt = sp.ntiles.cpu().numpy().astype(np.int64)
    rect = sp.rect.cpu().numpy().astype(np.int64)
    key = _sort_key(sp.dkey.cpu().numpy())
    tiles, recs = [], []
    for s, sensor in enumerate(rig.sensors):
        lidar = hasattr(sensor, "ray_az")
        cols = sensor.n_az_tiles if lidar else -(-sensor.width // sensor.tile_w)
        for r in np.nonzero(nt[s * n:(s + 1) * n])[0] + s * n:
            x0, y0, w, h = rect[r]
            t = (np.arange(y0, y0 + h)[:, None] * cols + (x0 + np.arange(w))[None, :] % cols).ravel()
            assert len(t) == nt[r]
            tiles.append(t + int(rig.tile_base[s] - rig.tile_base[0]))
            recs.append(np.full(len(t), r))
    tiles, recs = np.concatenate(tiles), np.concatenate(recs)
    order = np.lexsort((recs, key[recs], tiles))
    tiles, gid = tiles[order], recs[order] % n
    ends = np.searchsorted(tiles, np.arange(sp.n_tiles), side="right")
    starts = np.searchsorted(tiles, np.arange(sp.n_tiles), side="left")
    return nt, [gid[a:b].tolist() for a, b in zip(starts, ends)]


def _tied(g):
    """A third of the Gaussians in the places of others: equal depths, listed in the order of their ids."""
    n = len(g.means)
    g.means[: n // 3] = g.means[n - n // 3:][::-1]


@pytest.mark.parametrize("n,which", [(600, "c"), (2048, "c"), (4096, "l"), (8192, "c"), (8193, "l"), (4096, "cl"), (8192, "w")])
def test_equal_depths(n, which):
    b = _binding()
    g, cams, lids = _scene(n, 2.0, which)
    _tied(g)
    _check_lists(b, g, cams, lids, n)


@pytest.mark.parametrize("which", ["c", "l", "cl", "e", "wl"])
@pytest.mark.parametrize("n,size", [(1, 3.0), (63, 1.0), (130, 25.0), (2047, 1.0), (2049, 4.0), (4099, 0.3), (20011, 1.0)])
def test_lists(n, size, which):
    g, cams, lids = _scene(n, size, which)
    _check_lists(_binding(), g, cams, lids, n)


def _check_lists(b, g, cams, lids, n):
    rig = b.Rig(cams, lids)
    G = b.GaussTensors.from_numpy(g)
    sp = b.SensorPass(rig, 0, len(rig.sensors), n, 1, batched=len(rig.sensors) > 1)
    sp.fit_capacity(G, 1.1)
    for _ in range(2):   # the second pass meets the first one's records and scratch
        sp.status.zero_()
        sp.render(G)
    torch.cuda.synchronize()
    assert b.read_status(sp.status).overflow == 0
    if int((sp.ntiles > 0).sum()) == 0:
        assert all(not l for l in tile_lists_gpu(sp))
        return
    nt, lists = _expected(rig, sp, n)
    base = np.cumsum(nt) - nt
    np.testing.assert_array_equal(sp.entry_base.cpu().numpy()[nt > 0], base[nt > 0])
    assert tile_lists_gpu(sp) == lists
