"""hg_temporal_bwd without rows through the C ABI, where the context array may
be NULL whatever w is: the weight gradients are zero, or stay as they are with
accumulate = 1."""
import ctypes as C

import pytest

torch = pytest.importorskip("torch")

from paper_2608_02168_amd import api, synth
from tests.helpers import to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("accumulate", [0, 1])
@pytest.mark.parametrize("dtype", [api.HG_DTYPE_F32, api.HG_DTYPE_BF16])
@pytest.mark.parametrize("w", [0, 2, 4])
def test_no_rows_and_no_context_array(w, dtype, accumulate):
    p = {k: to_dev(v) for k, v in synth.temporal_weights(1, 64).items()}
    grads = {k: torch.full_like(v, 3.0) for k, v in p.items()}
    W = api.TemporalWeights(*[p[k].data_ptr() for k in api.TEMPORAL_PARAMS])
    G = api.TemporalWeights(*[grads[k].data_ptr() for k in api.TEMPORAL_PARAMS])
    ws = torch.empty(max(1, api.hg_temporal_bwd_workspace_size(0, 64, w)), dtype=torch.uint8, device="cuda")
    st = api.lib().hg_temporal_bwd(0, 64, w, dtype, None, None, C.byref(W), None, None, None, accumulate, C.byref(G),
                                   ws.data_ptr(), ws.numel(), torch.cuda.current_stream().cuda_stream)
    assert st == api.HG_OK, api.last_error_detail()
    torch.cuda.synchronize()
    for k, g in grads.items():
        assert torch.equal(g, torch.full_like(g, 3.0 * accumulate)), k
