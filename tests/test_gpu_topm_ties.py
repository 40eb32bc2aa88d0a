"""TopM over many candidates that share one key, small or large: the set is the
oracle's, and the search is over before its last launch, whose one block only
ranks the few composites left.  Walking 256 thousand candidates with its 256
threads takes a thousand dependent rounds of two loads each, half a millisecond
at half a microsecond a round, 2.9 ms for 1.5 million; ranking 256 takes some 10
us."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import select
from paper_2608_02168_amd import api

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [262_144, 262_145, 1_500_001])
@pytest.mark.parametrize("kind", ["small", "large", "largest", "two_values"])
def test_ties_of_many_candidates(kind, n):
    e, base, budget, seed = 2 * n, n // 50, n // 4, 9
    rng = np.random.default_rng(1)
    src, dst = rng.integers(0, n, e).astype(np.int32), rng.integers(0, n, e).astype(np.int32)
    part = (np.arange(n) >= base).astype(np.int32)
    # every node outside the base set is a candidate
    src[:n - base], dst[:n - base] = np.arange(base, n), 7
    keys = {"small": np.full(n, 3), "large": np.full(n, 2_000_000_000), "largest": np.full(n, 2**31 - 2),
            "two_values": np.where(np.arange(n) % 5 == 0, 2_050, 2_000_000_000)}[kind].astype(np.int32)
    t = [torch.from_numpy(x).cuda() for x in (src, dst, np.zeros(e, np.uint8), np.zeros(n, np.uint8), part)]
    k = torch.from_numpy(keys).cuda()
    api.hg_build_csr(*t, 0, 1, 1, budget, seed=seed, node_key=k)
    times = []
    for _ in range(3):
        api.hg_timing_enable(True)
        sub = api.hg_build_csr(*t, 0, 1, 1, budget, seed=seed, node_key=k)
        api.hg_timing_enable(False)
        launches, ms = api.hg_timing_collect()["build_select_finish"]
        assert launches == 1
        times.append(ms)
    ref = select.top_m(part == 1, keys.astype(np.int64), select.THETA_NONE, budget, seed)
    got = sub.view("local2global")[sub.view("overlap").long()].sort().values.cpu().numpy()
    assert np.array_equal(got, ref)
    assert min(times) < 0.25, times
