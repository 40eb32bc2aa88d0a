"""Backward work items of long CSC rows cut by destination blocks of 2^18
nodes: counts of the plan and parity of both backwards on both sides of one
and of two blocks, with rows at every edge of the cut (one entry under and at
24 entries a block, at and over one and two chunks a block).  Float32 against
the float64 oracle, element-wise relative error <= 1e-4 as for all layers."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import hgt, layer, select
from paper_2608_02168_amd import api, synth
from tests.helpers import pack_mask, parity_err, to_dev

pytestmark = pytest.mark.gpu
TOL = 1e-4
BLOCK, CHUNK, PIECE = 1 << 18, 64, 24  # fewer than 2^20 edges: chunks of 64


def _case(n, seed=5):
    """Hubs of the lengths where the cut changes, a light row for every 3rd node."""
    rng = np.random.default_rng(seed)
    b = -(-n // BLOCK)
    edges = sorted({PIECE * b - 1, PIECE * b, CHUNK, CHUNK + 1, CHUNK * b, CHUNK * b + 1, 2 * CHUNK * b,
                    2 * CHUNK * b + 1, 5000})
    hubs = rng.choice(n, len(edges), replace=False)
    light = np.arange(0, n, 3)
    src = np.concatenate([np.repeat(hubs, edges), light]).astype(np.int32)
    dst = rng.integers(0, n, src.size).astype(np.int32)
    rel = np.concatenate([np.repeat(np.arange(len(edges)) % 2, edges), light // 3 % 2]).astype(np.uint8)
    ntype = (np.arange(n) % 97 == 0).astype(np.uint8)
    part = np.zeros(n, dtype=np.int32)
    ref = select.build(src, dst, rel, ntype, part, 0, 2, 2, 0)
    sub = api.hg_build_csr(to_dev(src), to_dev(dst), to_dev(rel), to_dev(ntype), to_dev(part), 0, 2, 2, 0)
    assert ref.n_sub == sub.n_sub == n
    return b, ref, sub


def _expected_counts(b, csc_ptr):
    length = np.diff(csc_ptr)
    split = length[length > (CHUNK if b == 1 else PIECE * b - 1)]
    pieces = int((-(-split // (CHUNK * b)) * b).sum())
    return int((length > 0).sum()) - split.size + pieces, split.size, pieces


@pytest.mark.parametrize("n", [BLOCK, BLOCK + 1, 2 * BLOCK + 1])
def test_mean_backward(n):
    b, ref, sub = _case(n)
    assert (sub.c.plan_items, sub.c.plan_heavy, sub.c.plan_partials) == _expected_counts(b, ref.csc_ptr)
    d, rng = 64, np.random.default_rng(n)
    X, G = rng.normal(0, 1, (n, d)).astype(np.float32), rng.normal(0, 1, (n, d)).astype(np.float32)
    w = synth.layer_weights(3, 0, 2, 2, d, 0.1)
    mask = rng.random((n, d)) < 0.5
    exp = layer.backward(n, ref.src_l, ref.dst_l, ref.rel_l, ref.ntype_l, X, w.w_rel, w.w_self, w.bias, G, mask=mask)
    got = api.hg_layer_bwd(sub, to_dev(X), to_dev(w.w_rel), to_dev(w.w_self), to_dev(pack_mask(mask)), to_dev(G))
    for g, e, name in zip(got, exp, ("dH", "dW_rel", "dW_self", "dbias")):
        err = parity_err(g.cpu().numpy(), e)
        assert err <= TOL, (name, err)


@pytest.mark.parametrize("n", [BLOCK + 1])
def test_attention_backward(n):
    _, ref, sub = _case(n)
    d, heads, rng = 64, 4, np.random.default_rng(n)
    X, G = rng.normal(0, 1, (n, d)).astype(np.float32), rng.normal(0, 1, (n, d)).astype(np.float32)
    w = synth.hgt_weights(5, 0, 2, 2, d, heads, 0.1)
    p = hgt.Params(*[w[k] for k in hgt.PARAM_NAMES])
    wd = {k: to_dev(v) for k, v in w.items()}
    dH, grads = hgt.backward(n, ref.src_l, ref.dst_l, ref.rel_l, ref.ntype_l, X, p, heads, G,
                             mask=np.ones((n, d), dtype=bool))
    _, mask, saved = api.hg_hgt_fwd(sub, to_dev(X), wd, heads, relu=False)
    got, got_w = api.hg_hgt_bwd(sub, to_dev(X), wd, heads, mask, saved, to_dev(G), relu=False)
    err = parity_err(got.cpu().numpy(), dH)
    assert err <= TOL, err
    for k in hgt.PARAM_NAMES:
        err = parity_err(got_w[k].cpu().numpy(), getattr(grads, k))
        assert err <= TOL, (k, err)
