"""Which cut of the long CSC rows a plan takes: by destination blocks where it
has few pieces for its edges and leaves enough of them in whole rows, else by
length; counts on both sides of both bounds, in two blocks of destinations and
in nine, and all rows alike (the gradients in either cut are tested elsewhere)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2608_02168_amd import api

pytestmark = pytest.mark.gpu
BLOCK, CHUNK, PIECE = 1 << 18, 64, 24  # fewer than 2^20 edges: chunks of 64
TWO, NINE = BLOCK + 1, 8 * BLOCK + 1


def _plan(n, rows, light):
    """`rows`: entries of the first nodes' rows; `light` further rows of one entry."""
    src = np.concatenate([np.repeat(np.arange(len(rows)), rows), len(rows) + np.arange(light)]).astype(np.int32)
    dst = np.random.default_rng(len(rows)).integers(0, n, src.size).astype(np.int32)
    z = lambda k, t: torch.zeros(k, dtype=t, device="cuda")
    sub = api.hg_build_csr(torch.from_numpy(src).cuda(), torch.from_numpy(dst).cuda(), z(src.size, torch.uint8),
                           z(n, torch.uint8), z(n, torch.int32), 0, 1, 1, 0)
    assert (sub.n_sub, sub.e_sub) == (n, src.size)
    return sub.c.plan_items, sub.c.plan_heavy, sub.c.plan_partials


def _counts(rows, light, b):
    rows = np.asarray(rows)
    split = rows[rows > (PIECE * b - 1 if b > 1 else CHUNK)]
    size = np.maximum(CHUNK, np.minimum(1_024, split // 512))
    pieces = int((-(-split // (size * b)) * b).sum())
    return len(rows) - split.size + light + pieces, split.size, pieces


def _rule(rows, light, b):
    e = int(np.sum(rows)) + light
    split = np.asarray(rows)[np.asarray(rows) >= PIECE * b]
    pays = _counts(rows, light, b)[2] * (200 if b <= 8 else 100) <= e and 16 * split.sum() <= 15 * e
    return _counts(rows, light, b if pays else 1), pays


@pytest.mark.parametrize("n,rows,light,pays", [
    # pieces for the edges: 500 rows of 50 entries make 1000 pieces, 250 of 300 make 2250 in nine blocks
    (TWO, [50] * 500, 175_000, True), (TWO, [50] * 500, 174_999, False),
    (NINE, [300] * 250, 150_000, True), (NINE, [300] * 250, 149_999, False),
    # edges in split rows: 15 of 16
    (TWO, [600_500], 40_034, True), (TWO, [600_500], 40_033, False),
    # all rows alike, and nothing to split
    (TWO, [50] * 5_000, 0, False), (TWO, [47] * 300, 200_000, True), (BLOCK, [65] * 100, 100_000, False),
])
def test_cut_taken(n, rows, light, pays):
    expect, rule = _rule(rows, light, -(-n // BLOCK))
    if n > BLOCK:
        assert rule == pays
    assert _plan(n, rows, light) == expect
