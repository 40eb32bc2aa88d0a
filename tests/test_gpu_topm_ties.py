"""TopM over a million and more candidates that share one key, small or large:
the set is the oracle's, and the search is over before its last launch, whose
one block only ranks the few composites left.  Walking a million candidates
with its 256 threads takes 4000 dependent rounds of two loads each, over 2 ms
at half a microsecond a round; ranking 256 takes some 10 us."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import select
from paper_2608_02168_amd import api

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["small", "large", "largest", "two_values"])
def test_ties_of_a_million_candidates(kind):
    n, e, budget, seed = 1_500_001, 3_000_000, 400_003, 9
    rng = np.random.default_rng(1)
    src, dst = rng.integers(0, n, e).astype(np.int32), rng.integers(0, n, e).astype(np.int32)
    part = (np.arange(n) >= 400_000).astype(np.int32)
    # every node outside the base set is a candidate
    src[:n - 400_000], dst[:n - 400_000] = np.arange(400_000, n), 7
    keys = {"small": np.full(n, 3), "large": np.full(n, 2_000_000_000), "largest": np.full(n, 2**31 - 2),
            "two_values": np.where(np.arange(n) % 5 == 0, 2_050, 2_000_000_000)}[kind].astype(np.int32)
    t = [torch.from_numpy(x).cuda() for x in (src, dst, np.zeros(e, np.uint8), np.zeros(n, np.uint8), part)]
    k = torch.from_numpy(keys).cuda()
    api.hg_build_csr(*t, 0, 1, 1, budget, seed=seed, node_key=k)
    api.hg_timing_enable(True)
    sub = api.hg_build_csr(*t, 0, 1, 1, budget, seed=seed, node_key=k)
    api.hg_timing_enable(False)
    launches, ms = api.hg_timing_collect()["build_select_finish"]
    ref = select.top_m(part == 1, keys.astype(np.int64), select.THETA_NONE, budget, seed)
    got = sub.view("local2global")[sub.view("overlap").long()].sort().values.cpu().numpy()
    assert np.array_equal(got, ref)
    assert launches == 1 and ms < 1.0, ms
