"""Backward of rows that hold most of a small graph's edges: more pieces than a
row is cut into at the chunk of such a graph (64 and 256 entries), so that it
takes longer ones.  Counts of the plan and parity against the oracle, and the
time of adding up the partial rows, which one wave does row by row: some 600
pieces take tens of microseconds, the 8000 and 16000 of whole chunks 170 and
340 at d = 128."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import layer, select
from paper_2608_02168_amd import api, synth
from tests.helpers import pack_mask, parity_err, to_dev

pytestmark = pytest.mark.gpu
TOL = 1e-4  # element-wise relative error of float32 layers against the float64 oracle


@pytest.mark.parametrize("edges,chunk", [(1_000_000, 64), (1_100_000, 256)])
def test_star_backward(edges, chunk):
    n, d, hub = 20_000, 128, 17
    rng = np.random.default_rng(edges)
    src = np.full(edges, hub, dtype=np.int32)
    src[: n // 2] = np.arange(n // 2)
    dst = rng.integers(0, n, edges).astype(np.int32)
    rel, ntype, part = np.zeros(edges, np.uint8), np.zeros(n, np.uint8), np.zeros(n, np.int32)
    ref = select.build(src, dst, rel, ntype, part, 0, 1, 1, 0)
    sub = api.hg_build_csr(to_dev(src), to_dev(dst), to_dev(rel), to_dev(ntype), to_dev(part), 0, 1, 1, 0)
    length = np.diff(ref.csc_ptr)
    split = length[length > chunk]
    pieces = -(-split // np.maximum(chunk, np.minimum(1_024, split // 512)))
    assert (sub.c.plan_heavy, sub.c.plan_partials) == (split.size, pieces.sum())
    assert sub.c.plan_items == np.count_nonzero(length) - split.size + pieces.sum()
    assert pieces.max() > 500
    X, G = rng.normal(0, 1, (n, d)).astype(np.float32), rng.normal(0, 1, (n, d)).astype(np.float32)
    w = synth.layer_weights(3, 0, 1, 1, d, 0.1)
    mask = rng.random((n, d)) < 0.5
    exp = layer.backward(n, ref.src_l, ref.dst_l, ref.rel_l, ref.ntype_l, X, w.w_rel, w.w_self, w.bias, G, mask=mask)
    args = (sub, to_dev(X), to_dev(w.w_rel), to_dev(w.w_self), to_dev(pack_mask(mask)), to_dev(G))
    api.hg_layer_bwd(*args)
    times = []
    for _ in range(3):
        api.hg_timing_enable(True)
        got = api.hg_layer_bwd(*args)
        torch.cuda.synchronize()
        api.hg_timing_enable(False)
        times.append(api.hg_timing_collect()["spmm_bwd_reduce"][1])
    for g, e, name in zip(got, exp, ("dH", "dW_rel", "dW_self", "dbias")):
        err = parity_err(g.cpu().numpy(), e)
        assert err <= TOL, (name, err)
    assert min(times) < 0.1, times
