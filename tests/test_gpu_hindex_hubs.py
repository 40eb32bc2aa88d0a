"""h-indices of 4096 and more, which parallel edges to hubs give (an edge
counts its neighbour's out-degree each time): rows at the edges of the
histogram, of its ranges and of the walks that narrow them, bit-exact against
oracle.select, and the time of the longest row's walks: by parts they take
under a millisecond each, by one block once per 4096 values of h over a
second."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import select
from paper_2608_02168_amd import api

pytestmark = pytest.mark.gpu
HUB = 3_000_000  # neighbours of the longest row: ranges of 4096 degrees, two more walks


def _rows():
    """Out-neighbours of the first nodes, as (node, count) pairs; node 0 is the hub of self loops."""
    rows = [[(0, HUB)]]
    for n in (4_094, 4_095, 4_096, 4_097, 5_437, 5_438, 5_439, 5_440, 16_383, 16_384, 16_385, 50_000):
        rows.append([(0, n)])                    # h = n: every neighbour is the hub
    k = len(rows)
    rows.append([(0, 6_000)])                    # k: h = 6000
    rows.append([(0, 5_000), (k, 11_384)])       # one block: between two values
    rows.append([(0, 9_000), (k, 11_000)])       # by parts: above the lower value
    rows.append([(k + 2, 40_000), (0, 10_000), (k, 50_000)])
    rows.append([(0, 4_095), (k, 1), (k + 9, 20_000)])
    rows.append([(0, 1_000_000), (k + 3, 2_000_000)])
    return rows


def _graph():
    rng = np.random.default_rng(4)
    n, src, dst = 60_001, [], []
    for v, row in enumerate(_rows()):
        for u, c in row:
            src.append(np.full(c, v))
            dst.append(np.full(c, u))
    src.append(rng.integers(0, n, 200_000))
    dst.append(rng.integers(0, n, 200_000))
    src, dst = np.concatenate(src), np.concatenate(dst)
    order = rng.permutation(src.size)
    return n, src[order].astype(np.int32), dst[order].astype(np.int32)


def test_high_h_index():
    n, src, dst = _graph()
    ref = select.out_hindex(n, src, dst)
    assert ref[0] >= HUB and np.count_nonzero(ref >= 4_096) >= 15
    s, d = torch.from_numpy(src).cuda(), torch.from_numpy(dst).cuda()
    rel = torch.zeros(src.size, dtype=torch.uint8, device="cuda")
    times = []
    for _ in range(2):
        api.hg_timing_enable(True)
        got = api.hg_node_keys(s, d, rel, n, 1, api.HG_KEY_HINDEX)
        api.hg_timing_enable(False)
        times.append(sum(t for k, (_, t) in api.hg_timing_collect().items() if k.startswith("hindex")))
    assert np.array_equal(got.cpu().numpy(), ref)
    assert min(times) < 50, times
    part = (np.arange(n) >= 30_000).astype(np.int32)
    nt, p = torch.zeros(n, dtype=torch.uint8, device="cuda"), torch.from_numpy(part).cuda()
    for theta in (3, 4_095, 4_096, 5_500, select.THETA_NONE):
        sub = api.hg_build_csr(s, d, rel, nt, p, 1, 1, 1, 20_000, key=api.HG_KEY_HINDEX, theta=theta, seed=5)
        over = sub.view("local2global")[sub.view("overlap").long()].sort().values.cpu().numpy()
        assert np.array_equal(over, select.top_m(select.candidates(part, 1, src, dst), ref, theta, 20_000, 5)), theta
