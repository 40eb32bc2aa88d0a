"""hg_build_csr at the edges of its tiles and of its selection digits: long
stretches of rows without entries, node counts around the tile sizes, 255
relations, split rows, and caller-given keys of every width, bit-exact against
oracle.select."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import select
from paper_2608_02168_amd import api
from tests.test_gpu_build import assert_same

pytestmark = pytest.mark.gpu


def _dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


def _graph(n, e, n_rel, n_ntype, seed, src_ids=None, dst_ids=None):
    rng = np.random.default_rng(seed)
    src = (rng.integers(0, n, e) if src_ids is None else rng.choice(src_ids, e)).astype(np.int32)
    dst = (rng.integers(0, n, e) if dst_ids is None else rng.choice(dst_ids, e)).astype(np.int32)
    rel = rng.integers(0, n_rel, e).astype(np.uint8)
    ntype = rng.integers(0, n_ntype, n).astype(np.uint8)
    part = (rng.random(n) < 0.3).astype(np.int32)
    return src, dst, rel, ntype, part


def _chunks(lengths, limit, size):
    nch = -(-lengths // size)
    return nch, nch[lengths > limit]


# (nodes, edges, relations, node types, source ids, destination ids)
SHAPES = {
    "few_sources": (70_001, 5_000, 3, 2, [0, 1, 2, 69_999], None),
    "few_destinations": (70_001, 9_000, 3, 2, None, [7, 50_000]),
    "one_edge": (300_000, 1, 5, 2, [123], [299_999]),
    "one_node": (1, 40, 2, 1, None, None),
    "tile_256": (256, 4_000, 4, 2, None, None),
    "tile_257": (257, 4_000, 4, 2, [5, 256], None),
    "tile_2048": (2_048, 30_001, 1, 2, None, None),
    "tile_2049": (2_049, 30_001, 7, 1, None, [2_048]),
    "rel_255": (2_100, 50_000, 255, 2, None, None),
    "three_types": (4_097, 40_000, 5, 3, None, None),
    "edges_below_2_20": (5_000, (1 << 20) - 1, 3, 2, None, None),
    "edges_2_20": (5_000, 1 << 20, 3, 2, None, None),
}


@pytest.mark.parametrize("name", sorted(SHAPES))
def test_build_shapes(name):
    n, e, n_rel, n_ntype, src_ids, dst_ids = SHAPES[name]
    src, dst, rel, ntype, part = _graph(n, e, n_rel, n_ntype, 11, src_ids, dst_ids)
    budget = max(1, n // 9)
    ref = select.build(src, dst, rel, ntype, part, 0, n_rel, n_ntype, budget, 0, select.THETA_NONE, 3)
    sub = api.hg_build_csr(_dev(src), _dev(dst), _dev(rel), _dev(ntype), _dev(part), 0, n_rel, n_ntype, budget, seed=3)
    assert_same(ref, sub)
    # the plan's counts: chunks of a size by the edges per CSC row, of 2048 per destination row above 2048 entries
    length = np.diff(ref.csc_ptr)
    chunk = 64 if e < 1 << 20 else (256 if e < 1 << 23 else 1024)
    nch, split = _chunks(length, chunk, chunk)
    assert (sub.c.plan_items, sub.c.plan_heavy, sub.c.plan_partials) == (nch.sum(), split.size, split.sum())
    into = np.add.reduceat(np.diff(ref.csr_ptr), np.arange(0, ref.n_sub * n_rel, n_rel)) if ref.n_sub else length[:0]
    _, fsplit = _chunks(into, 2048, 2048)
    assert (sub.c.plan_fwd_heavy, sub.c.plan_fwd_parts) == (fsplit.size, fsplit.sum())


def _keys(kind, n, rng):
    if kind == "equal_small":
        return np.full(n, 3)
    if kind == "equal_large":
        return np.full(n, 2_000_000_000)
    if kind == "edge_of_small":
        return rng.integers(2045, 2050, n)
    if kind == "two_values":
        return np.where(rng.random(n) < 0.4, 7, 1 << 22)
    return rng.integers(0, 2**31 - 1, n)


@pytest.mark.parametrize("budget", [0, 1, 1_025, 9_000, 10**6])
@pytest.mark.parametrize("kind", ["equal_small", "equal_large", "edge_of_small", "two_values", "wide"])
def test_selection_by_given_keys(kind, budget):
    """The digits of the search: keys below and above its first digit, ranges
    that end in the key and in the hash, everything and nothing taken."""
    n, e = 30_011, 200_000
    src, dst, rel, ntype, part = _graph(n, e, 2, 2, 5)
    keys = _keys(kind, n, np.random.default_rng(6)).astype(np.int32)
    theta = select.THETA_NONE
    ref = select.top_m(select.candidates(part, 1, src, dst), keys.astype(np.int64), theta, budget, 77)
    sub = api.hg_build_csr(_dev(src), _dev(dst), _dev(rel), _dev(ntype), _dev(part), 1, 2, 2, budget, seed=77,
                           node_key=_dev(keys))
    assert sub.m_sel == ref.size
    got = sub.view("local2global")[sub.view("overlap").long()].sort().values.cpu().numpy()
    assert np.array_equal(got, ref)


def _hindex_graph(name):
    """Edges whose out-neighbour lists have the lengths where the h-index
    changes its way: 16 / 17, 1024 / 1025, 16384 / 16385 neighbours, several
    parts, and an h-index past 4096 (a dense core of 4500 nodes)."""
    rng = np.random.default_rng(9)
    n = 30_001
    if name == "lengths":
        lengths = [0, 1, 2, 15, 16, 17, 63, 64, 65, 1_023, 1_024, 1_025, 5_000, 16_384, 16_385, 40_000]
        src = np.repeat(np.arange(len(lengths)) * 1_700 + 3, lengths)
        src = np.concatenate([src, rng.integers(0, n, 90_000)])  # degrees of the neighbours
        dst = rng.integers(0, n, src.size)
    else:
        core = 4_500
        a = np.arange(core)
        src = np.concatenate([np.repeat(a, core), rng.integers(0, n, 50_000)])
        dst = np.concatenate([np.tile(a, core), rng.integers(0, n, 50_000)])
    order = rng.permutation(src.size)
    return n, src[order].astype(np.int32), dst[order].astype(np.int32)


@pytest.mark.parametrize("name", ["lengths", "core"])
def test_hindex_lengths(name):
    n, src, dst = _hindex_graph(name)
    rel = np.zeros(src.size, np.uint8)
    ref = select.out_hindex(n, src, dst)
    got = api.hg_node_keys(_dev(src), _dev(dst), _dev(rel), n, 1, api.HG_KEY_HINDEX).cpu().numpy()
    assert np.array_equal(got, ref)
    part = (np.arange(n) % 3 == 0).astype(np.int32)
    cand = select.candidates(part, 1, src, dst)
    ntype = np.zeros(n, np.uint8)
    for theta, budget in ((2, 500), (select.THETA_NONE, 4_000)):
        sub = api.hg_build_csr(_dev(src), _dev(dst), _dev(rel), _dev(ntype), _dev(part), 1, 1, 1, budget,
                               key=api.HG_KEY_HINDEX, theta=theta, seed=5)
        over = sub.view("local2global")[sub.view("overlap").long()].sort().values.cpu().numpy()
        assert np.array_equal(over, select.top_m(cand, ref, theta, budget, 5))


def test_hindex_range_error():
    n = 5_000
    src = np.arange(n, dtype=np.int32)
    dst = np.arange(n, dtype=np.int32)[::-1].copy()
    rel, z = np.zeros(n, np.uint8), np.zeros(n, np.uint8)
    for bad in (-1, n, 2**31 - 1):
        s = src.copy()
        s[1_234] = bad
        with pytest.raises(api.HgError):
            api.hg_node_keys(_dev(s), _dev(dst), _dev(rel), n, 1, api.HG_KEY_HINDEX)
        with pytest.raises(api.HgError):
            api.hg_build_csr(_dev(s), _dev(dst), _dev(rel), _dev(z), _dev(z.astype(np.int32)), 0, 1, 1, 7,
                             key=api.HG_KEY_HINDEX)
