"""Weight gradients of more products than one launch's partial rows hold (8192,
4096 and 1024 at d = 64, 128 and 256, 512 a product of 262144 rows and more), so
that a batch runs in parts, and of more than its 24 products; overwritten and
added into, against float64 products by plain torch (1e-4 of the value or the
RMS for float32, 2e-2 for bfloat16)."""
import pytest

torch = pytest.importorskip("torch")

from paper_2608_02168_amd import api, synth

pytestmark = pytest.mark.gpu
N = 263_000


def _err(got, ref):
    return float(((got.double() - ref).abs() / torch.maximum(ref.abs(), ref.pow(2).mean().sqrt())).max())


# width, storage, relations with an edge of every node, node types
@pytest.mark.parametrize("d,dtype,R,T", [
    (64, "f32", 17, 1), (128, "f32", 9, 2), (256, "f32", 3, 1), (256, "bf16", 3, 1), (128, "bf16", 9, 1),
    (64, "f32", 26, 26), (256, "f32", 1, 3)])
def test_batches_in_parts(d, dtype, R, T):
    n = N * T if (R, T) == (1, 3) else N  # types of 263000 rows each, or relations
    g = torch.Generator(device="cuda")
    g.manual_seed(d + R)
    src = torch.arange(n, device="cuda", dtype=torch.int32).repeat(R)
    rel = torch.arange(R, device="cuda").repeat_interleave(n).to(torch.uint8)
    dst = torch.randint(0, n, src.shape, generator=g, device="cuda", dtype=torch.int32)
    ntype = (torch.arange(n, device="cuda") * T // n).to(torch.uint8)  # types in id order: local ids are the ids
    sub = api.hg_build_csr(src, dst, rel, ntype, torch.zeros(n, dtype=torch.int32, device="cuda"), 0, R, T, 0,
                           want_eid=False)
    assert sub.n_sub == n and sub.n_active() == [n] * R
    dt, tol = (torch.float32, 1e-4) if dtype == "f32" else (torch.bfloat16, 2e-2)
    H = torch.randn((n, d), generator=g, device="cuda").to(dt)
    G = torch.randn((n, d), generator=g, device="cuda").to(dt)
    w = synth.layer_weights(3, 0, R, T, d, 0.0)
    W_rel, W_self = torch.from_numpy(w.w_rel).cuda(), torch.from_numpy(w.w_self).cuda()
    mask = torch.full((n, d // 32), -1, dtype=torch.int32, device="cuda")
    H64, G64 = H.double(), G.double()
    ref_rel = torch.empty((R, d, d), dtype=torch.float64, device="cuda")
    for r in range(R):
        t = dst[r * n:(r + 1) * n].long()
        dY = G64[t] / torch.bincount(t, minlength=n).double()[t, None]  # one edge of every source, in order
        ref_rel[r] = H64.T @ dY
    off = sub.type_off_host()
    ref_self = torch.stack([H64[off[k]:off[k + 1]].T @ G64[off[k]:off[k + 1]] for k in range(T)])
    ref_bias = torch.stack([G64[off[k]:off[k + 1]].sum(0) for k in range(T)])
    ws = torch.empty(api.hg_layer_bwd_workspace_size(sub, d, dt), dtype=torch.uint8, device="cuda")
    out = [torch.full(x.shape, float("nan"), device="cuda") for x in (ref_rel, ref_self, ref_bias)]
    for accumulate in (False, True):
        start = [x.clone() for x in out]
        api.hg_layer_bwd(sub, H, W_rel, W_self, mask, G, dW_rel=out[0], dW_self=out[1], dbias=out[2], ws=ws,
                         accumulate=accumulate)
        for got, s, ref, what in zip(out, start, (ref_rel, ref_self, ref_bias), ("dW_rel", "dW_self", "dbias")):
            err = _err(got, ref + s.double() if accumulate else ref)
            assert err <= tol, (what, accumulate, err)
