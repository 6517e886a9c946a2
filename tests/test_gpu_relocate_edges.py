"""Relocation at the edges of its draw: the sizes where the samples' spacing changes (2^15, 2^16, ...: none
to two 8-way levels below them), runs without weight across a sample, all but the first or last Gaussian
dead, and rows of the smallest and of more than 16 features, against the oracle (targets and copies bit
for bit, the bars of test_gpu_relocate.py otherwise)."""
import numpy as np
import pytest
import torch

from oracle import mcmc
from test_gpu_relocate import _binding, _check, _run, _scene

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [2, 8, 255, 4097, 32768, 32769, 65537, 131073, 262145])
@pytest.mark.parametrize("dead", [0.05, 0.7])
def test_sample_spacing(n, dead):
    g, u = _scene(3 * n, n, dead)
    G, tgt, moved = _run(_binding(), g, u)
    assert moved == int((g.opacities <= np.float32(0.005)).sum())
    _check(G, tgt, g, u)


@pytest.mark.parametrize("alive", [[0], [39_999], [0, 39_999], [4095, 4096, 20_000], list(range(8190, 8200))])
def test_long_runs_without_weight(alive):
    n = 40_000
    g, u = _scene(5, n, 1.0)
    g.opacities[alive] = np.linspace(0.3, 0.9, len(alive)).astype(np.float32)
    u[:4] = (0, 1, 0xFFFFFFFF, 0x80000000)
    G, tgt, moved = _run(_binding(), g, u)
    assert moved == n - len(alive)
    _check(G, tgt, g, u)


@pytest.mark.parametrize("n_feat", [3, 16, 17, 40])
def test_feature_rows(n_feat):
    g, u = _scene(n_feat, 5000, 0.3, n_feat=n_feat)
    G, tgt, _ = _run(_binding(), g, u)
    _check(G, tgt, g, u)


def test_rows_without_velocities():
    b = _binding()
    g, u = _scene(2, 3000, 0.4)
    ref, rt = mcmc.relocate(g, u)
    G = b.GaussTensors.from_numpy(g)
    G.velocities = None
    tgt, _ = b.mcmc_relocate(G, torch.from_numpy(u.astype(np.uint32).view(np.int32)).cuda())
    torch.cuda.synchronize()
    np.testing.assert_array_equal(tgt.cpu().numpy(), rt)
    np.testing.assert_array_equal(G.means.cpu().numpy(), ref.means)
    np.testing.assert_array_equal(G.quats.cpu().numpy(), ref.quats)
    np.testing.assert_array_equal(G.features.cpu().numpy(), ref.features)
