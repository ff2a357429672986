"""The wavefront traversal of yarn scenes (a quad of lanes per ray, subtrees
and samples shared among a wavefront's lanes) where its batching can go wrong:
ray counts around its batches of 16 and 32 rays and around the count from
which a wavefront takes 32, a bundle whose rays list more than 64 candidate
spans at once, and rays that skim a weave and share their subtrees.  Hits are
compared with the FP64 intersection oracle, and a ray's hit must not depend on
the rays traced with it."""
import numpy as np
import pytest

import oracle
from paper_2401_12724_amd import bysdf, workloads as W
from test_gpu_scene import _compare, _run

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return torch


def _bundle(n_yarns=40, seed=5):
    """Nearly parallel yarns along x whose tubes overlap, gently bent."""
    rng = np.random.default_rng(seed)
    x = np.linspace(-1.0, 1.0, 24)
    ctrl, off = [], [0]
    for _ in range(n_yarns):
        y0, z0, ph = rng.uniform(-0.1, 0.1), rng.uniform(-0.1, 0.1), rng.uniform(0, 6.28)
        y, z = y0 + 0.02 * np.sin(2.0 * x + ph), z0 + 0.02 * np.cos(1.5 * x + ph)
        ctrl.append(np.stack([x, y, z, np.full_like(x, 0.05)], 1))
        off.append(off[-1] + len(x))
    return np.concatenate(ctrl).astype(np.float32), np.array(off, np.int64), \
        np.zeros(n_yarns, np.int32), rng.uniform(0, 6.28, n_yarns).astype(np.float32)


@pytest.mark.parametrize("n", [1, 15, 16, 17, 31, 33, 47, 64, 65, 1000])
def test_bundle_batch_edges(torch_cuda, n):
    torch = torch_cuda
    ctrl, off, ty, ph = _bundle()
    S = bysdf.yarn_scene_create(ctrl, off, ty, ph)
    o, d = W.random_rays(n, 100 + n, (-0.9, -0.6, 0.3), (0.9, 0.6, 0.7), (-0.9, -0.1, -0.1), (0.9, 0.1, 0.1))
    tm = np.full(n, 50.0, np.float32)
    g = _run(torch, S, o, d, tm)
    _compare(g, oracle.intersect(oracle.Scene(ctrl, off), o, d, tm, 1e-4), ph, "bundle %d" % n)


def test_skimming_rays(torch_cuda):
    """Rays along the top of a weave: hundreds of nodes each, few hits."""
    torch = torch_cuda
    ctrl, off, ty, ph = W.weave(40, 40)
    S = bysdf.yarn_scene_create(ctrl, off, ty, ph)
    rng = np.random.default_rng(8)
    n = 300
    o = np.stack([np.full(n, -3.5), rng.uniform(-2.5, 2.5, n), rng.uniform(0.055, 0.085, n)], 1).astype(np.float32)
    t = np.stack([np.full(n, 3.5), rng.uniform(-2.5, 2.5, n), rng.uniform(0.055, 0.085, n)], 1)
    d = t - o
    d = (d / np.linalg.norm(d, axis=1, keepdims=True)).astype(np.float32)
    tm = np.full(n, 100.0, np.float32)
    g = _run(torch, S, o, d, tm)
    _compare(g, oracle.intersect(oracle.Scene(ctrl, off), o, d, tm, 1e-4), ph, "skimming")


@pytest.mark.parametrize("n", [131071, 131072, 131107])
def test_hit_independent_of_batch(torch_cuda, n):
    """Wavefronts take 16 rays below 131,072 and 32 from there on; the same
    rays in batches of 4,111 give the same bytes."""
    torch = torch_cuda
    ctrl, off, ty, ph = W.weave(24, 24)
    S = bysdf.yarn_scene_create(ctrl, off, ty, ph)
    o, d = W.random_rays(n, 9, (-2, -2, 0.05), (2, 2, 1.0), (-2, -2, -0.05), (2, 2, 0.05))
    tm = np.full(n, 1e3, np.float32)
    g = _run(torch, S, o, d, tm)
    for a in (0, 65536, n - 4111):
        b = a + 4111
        p = _run(torch, S, o[a:b], d[a:b], tm[a:b])
        for k in g:
            assert np.array_equal(g[k][a:b], p[k]), (k, a)
