"""A launch repeated on the same inputs gives the same bytes: every query
entry point over the largest types (8 plies, 16 nodes, 8 migration tables)
and over mixed types, in mixed and in type order, with other kernels launched
in between.  The queries' results do not depend on each other, so there is
nothing for an order of execution to change."""
import numpy as np
import pytest

from paper_2401_12724_amd import bysdf, workloads as W

from test_gpu_limits import _largest_types
from test_gpu_parity import _hetero_types

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ordered", [False, True])
@pytest.mark.parametrize("types", ["largest", "mixed"])
def test_launches_repeat(types, ordered):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    P = _largest_types() if types == "largest" else _hetero_types(43)
    nt, n = len(P), 16384 + 41
    tid = np.sort(np.random.default_rng(3).integers(0, nt, n)).astype(np.int32)
    q = W.queries(n, 17, type_ids=tid, v_max=40.0, with_xi=True) if ordered else \
        W.queries(n, 17, n_types=nt, v_max=40.0, with_xi=True)
    T, qd = bysdf.bysdf_types_create(P), bysdf.to_device(W.footprints(q, 5))
    qs = {k: a for k, a in qd.items() if k != "xi"}  # the library's own draws
    ops = [lambda: bysdf.bysdf_eval(T, qd), lambda: bysdf.bysdf_sample_pdf(T, qd),
           lambda: bysdf.bysdf_sample_pdf(T, qs), lambda: bysdf.bysdf_eval_sample(T, qd),
           lambda: bysdf.bysdf_eval_multi(T, qd, 16), lambda: bysdf.bysdf_sample_multi(T, qd, 16),
           lambda: bysdf.bysdf_sample_multi(T, qs, 16), lambda: bysdf.bysdf_ply_geometry(T, qd)]
    if ordered:
        off = np.concatenate([[0], np.cumsum(np.bincount(tid, minlength=nt))]).astype(np.int64)
        offd = torch.from_numpy(off).cuda()
        gE = torch.from_numpy(np.random.default_rng(4).normal(size=(n, 3)).astype(np.float32)).cuda()
        ops += [lambda: bysdf.bysdf_eval_batched(T, offd, qd),
                lambda: bysdf.bysdf_eval_backward(T, qd, offd, gE, per_query=True)]
    first = [[x.contiguous().view(torch.int32).clone() for x in f()] for f in ops]
    for _ in range(4):
        for k, f in enumerate(ops):
            for a, b in zip(first[k], f()):
                assert torch.equal(a, b.contiguous().view(torch.int32)), k
