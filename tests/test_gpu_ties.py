"""Rays whose closest entry is shared by several spans to the last bit: rays at
the joints of straight yarns, and yarns laid exactly on others.  Which span is
reported must not depend on the rays traced with it nor on how many spans its
wavefront meets."""
import numpy as np
import pytest

from paper_2401_12724_amd import bysdf
from test_gpu_scene import _run

pytestmark = pytest.mark.gpu


def _stack(n_yarns, copies, points=64):
    """Straight yarns along x, tops within 0.1 R of each other, each laid
    `copies` times; the joints between spans are at multiples of 1/16."""
    rng = np.random.default_rng(7)
    x = (np.arange(points) - points // 2) / 16.0
    ctrl, off = [], [0]
    for k in range(n_yarns):
        y, z = rng.integers(-8, 9) / 8192.0, rng.integers(-8, 9) / 8192.0
        for _ in range(copies):
            ctrl.append(np.stack([x, np.full_like(x, y), np.full_like(x, z), np.full_like(x, 0.0625)], 1))
            off.append(off[-1] + points)
    return (np.concatenate(ctrl).astype(np.float32), np.array(off, np.int64), np.zeros(len(off) - 1, np.int32),
            np.zeros(len(off) - 1, np.float32))


@pytest.mark.parametrize("n_yarns,copies", [(1, 1), (3, 1), (48, 1), (24, 3)])
def test_ties_independent_of_batch(n_yarns, copies):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    S = bysdf.yarn_scene_create(*_stack(n_yarns, copies))
    n = 160
    rng = np.random.default_rng(11)
    o = np.stack([rng.integers(-24, 25, n) / 16.0, rng.integers(-4, 5, n) / 1024.0, np.full(n, 1.0)], 1).astype(np.float32)
    d = np.tile(np.float32([0, 0, -1]), (n, 1))
    tm = np.full(n, 10.0, np.float32)
    g = _run(torch, S, o, d, tm)
    assert np.all(g["yarn"] >= 0)
    at = np.concatenate([[i, i + 1] for i in range(0, n, 7)])[:48]
    for i in at:
        p = _run(torch, S, o[i:i + 1], d[i:i + 1], tm[i:i + 1])
        for k in g:
            assert np.array_equal(g[k][i:i + 1], p[k]), (k, i)
    # among other rays, in another order
    order = rng.permutation(n)
    p = _run(torch, S, o[order], d[order], tm[order])
    for k in g:
        assert np.array_equal(g[k][order], p[k]), k


def test_ties_inside_a_bundle():
    """Rays that start within a bundle of overlapping yarns: their origins lie
    in several boxes at once, at equal distances."""
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    rng = np.random.default_rng(2)
    x = np.linspace(-1.0, 1.0, 24)
    ctrl = np.concatenate([np.stack([x, rng.uniform(-.1, .1) + 0.02 * np.sin(2 * x),
                                     rng.uniform(-.1, .1) + 0.02 * np.cos(1.5 * x), np.full_like(x, .05)], 1)
                           for _ in range(40)]).astype(np.float32)
    S = bysdf.yarn_scene_create(ctrl, np.arange(41, dtype=np.int64) * 24, np.zeros(40, np.int32),
                                np.zeros(40, np.float32))
    n = 200003
    o = (rng.uniform(-1, 1, (n, 3)) * [1, .12, .12]).astype(np.float32)
    d = rng.normal(size=(n, 3)).astype(np.float32)
    tm = np.full(n, 50.0, np.float32)
    g = _run(torch, S, o, d, tm)
    order = rng.permutation(n)
    p = _run(torch, S, o[order], d[order], tm[order])
    for k in g:
        assert np.array_equal(g[k][order], p[k]), k
