"""Gradients of tied weights in one buffer: with accumulate = 1 it collects the
sum of the gradients named for it, one after another, and with accumulate = 0
the last of them; both exact against the gradients in buffers of their own."""
import pytest

torch = pytest.importorskip("torch")

from paper_2608_02168_amd import api, synth
from tests.helpers import to_dev
from tests.test_gpu_hgt import CFGS, dev_weights, setup
from tests.test_gpu_temporal import case

pytestmark = pytest.mark.gpu


def _check(run, order, tied):
    """run(grads, accumulate) fills a dict of gradient buffers; `tied` names share one, `order` is the
    order in which the library adds them."""
    own = run({}, False)
    for accumulate in (True, False):
        start = {k: torch.randn_like(v) for k, v in own.items()}
        for k in tied:
            start[k] = start[tied[0]]
        expect = start[tied[0]].clone()
        for k in order:
            if k in tied:
                expect = expect + own[k] if accumulate else own[k]
        got = run(start, accumulate)
        assert torch.equal(got[tied[0]], expect), (tied, accumulate)


@pytest.mark.parametrize("name", ["tiny_d64_h4", "tiny_d128_h4"])
@pytest.mark.parametrize("tied", [("W_K", "W_V"), ("W_Q", "W_V"), ("W_K", "W_Q", "W_V"), ("W_agg", "W_K"),
                                  ("b_K", "b_V")])
def test_attention(name, tied):
    cfg, d, heads = CFGS[name]
    ref, sub, X, w = setup(cfg, d, heads)
    Xd, wd, G = to_dev(X), dev_weights(w), to_dev(synth.upstream_grad(3, ref.n_sub, d))
    _, mask, saved = api.hg_hgt_fwd(sub, Xd, wd, heads)

    def run(grads, accumulate):
        grads = grads or {k: torch.empty_like(v) for k, v in wd.items()}
        return api.hg_hgt_bwd(sub, Xd, wd, heads, mask, saved, G, grads=grads, accumulate=accumulate)[1]

    _check(run, ("W_agg", "W_K", "W_Q", "W_V", "b_agg", "b_K", "b_Q", "b_V"), tied)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("tied", [("Wi", "Wh"), ("bi", "bh")])
def test_temporal(tied, dtype):
    h, C, p, dH = case(7, 1_000, 2)
    hd, dHd, Cd = to_dev(h).to(dtype), to_dev(dH).to(dtype), [to_dev(c).to(dtype) for c in C]
    W = {k: to_dev(v) for k, v in p.items()}

    def run(grads, accumulate):
        grads = grads or {k: torch.empty_like(v) for k, v in W.items()}
        return api.hg_temporal_bwd(hd, Cd, W, dHd, grads=grads, accumulate=accumulate)[1]

    _check(run, ("Wi", "Wh", "bi", "bh"), tied)
