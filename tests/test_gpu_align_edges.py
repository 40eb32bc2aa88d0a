"""The alignment's Gram pass at the edges of its steps (32 rows), of its
smallest chunk (64 rows) and of the chunk count (448 chunks of 64 rows at
d = 128, 128 at d = 256), against the oracle at the bars of the alignment's
other tests (1e-4 for float32, 2e-2 for bfloat16)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import align
from paper_2608_02168_amd import api, synth
from tests.helpers import parity_err, to_dev
from tests.test_gpu_align import make

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("d", [64, 128, 256])
@pytest.mark.parametrize("m", [32, 63, 64, 65, 8_193, 28_672, 28_673])
def test_align_edges(m, d, dtype):
    bar, dt = (1e-4, torch.float32) if dtype == "f32" else (2e-2, torch.bfloat16)
    H, ov, Href = make(2 * m + 11, m, d, seed=m + d)
    if dtype == "bf16":
        H, Href = synth.round_bf16(H), synth.round_bf16(Href)
    (li, ld, L), dX, dY = align.loss_and_grad(H[ov], Href)
    dH = torch.zeros(H.shape, dtype=dt, device="cuda")
    dHref = torch.empty((m, d), dtype=dt, device="cuda")
    loss = api.hg_align_loss_fwd_bwd(to_dev(H).to(dt), to_dev(ov), to_dev(Href).to(dt), dH, dH_ref=dHref).cpu().numpy()
    for got, exp in zip(loss, (li, ld, L)):
        assert abs(got - exp) <= 1e-4 * abs(exp)
    got = dH.float().cpu().numpy()
    assert parity_err(got[ov], dX) <= bar
    assert not got[np.setdiff1d(np.arange(H.shape[0]), ov)].any()
    assert parity_err(dHref.float().cpu().numpy(), dY) <= bar
