"""Preparation of the CSR product: matrices of up to three rows per entry take one launch that works tile by tile, the
others the launches over the rows.  Compared with the oracle where the first can go wrong: rows across tiles and at their
borders, runs of empty rows, tiles with so many rows that several workgroups share them, both sides of the rule, a workspace full of garbage.  Whole numbers, sums below 2^24: every
result is exact."""
import numpy as np
import pytest
import torch

import oracle
from paper_2506_23906_amd import binding as B
from parity_util import dev

pytestmark = pytest.mark.gpu
ROUND = 2048         # rows that a workgroup looks at in a round
SHARE = 8192         # rows of a piece of a tile that several workgroups share


def lengths_of(kind, tile):
    rng = np.random.default_rng(41)
    if kind == "one row":
        return np.array([8])
    if kind == "one row of many tiles":
        return np.array([3 * tile + 5])
    if kind == "starts at tile borders":               # a row per tile; one that ends at the border, one that ends behind it
        return np.array([tile, tile, tile - 1, 2, tile - 1, 2 * tile, 100])
    if kind == "empty rows around":                    # leading, trailing, and at a border of two tiles
        return np.r_[np.zeros(3000, int), tile - 7, np.zeros(ROUND + 1, int), 7, np.zeros(ROUND, int), tile, np.zeros(9, int),
                     tile // 2, np.zeros(ROUND - 1, int), 400_000, np.zeros(5000, int)]
    if kind == "long runs of empty rows":              # of lengths around what a workgroup looks at in a round
        runs = [1, ROUND - 2, ROUND - 1, ROUND, ROUND + 1, 2 * ROUND - 1, 2 * ROUND, 2 * ROUND + 1, 3 * ROUND + 77, 1, 1]
        return np.concatenate([np.r_[np.zeros(k, int), 200_000 + 31 * k] for k in runs])
    if kind == "last row of a round":                  # all rows in the first tile: a full round, then up to the end of one
        return np.r_[np.ones(300, int), np.zeros(ROUND - 301, int), 5, 1, np.zeros(ROUND - 2, int), 17, 0, 1, 16 * ROUND + 50_000]
    if kind == "almost empty rows":                    # searched for by position: far apart, adjacent, at the borders of words
        a = np.zeros(200_000, int)
        a[[3, 4, 5, 700, 4000, 4001, 70_000, 199_999]] = [30, 1, 1, 31, 1, 64, 1900, 1]
        a[100_000:130_000:97] = 5
        return np.r_[tile + 17, a, 500_000]
    if kind == "rows of a wave":                       # borders of 64 rows and of a wave's share
        return np.r_[[int(i % 64 in (0, 63) or i % 1024 in (1, 1022)) for i in range(5000)], 50_000]
    if kind == "some tiles with empty rows":
        a = rng.integers(1, 60, 6000)
        b = np.where(rng.random(6000) < 0.3, 0, rng.integers(1, 60, 6000))
        return np.r_[a, b, a[::-1], b]
    if kind == "zipf":
        return np.minimum(rng.zipf(1.4, 30_000), 9000) + 3
    if kind == "sorted by degree":                     # nearly all rows in the last tiles, one in 20 of one entry
        tail = np.zeros(300_000, int)
        tail[rng.choice(300_000, 15_000, replace=False)] = 1
        return np.r_[np.sort(rng.zipf(1.3, 2000) % 3000)[::-1], rng.integers(8, 24, 4000), tail]
    if kind == "rows of many tiles among empty ones":  # shared tiles with one start or none of their own
        return np.concatenate([np.r_[np.zeros(20_000 + 13 * i, int), 6 * tile + 100 * i] for i in range(4)] + [np.zeros(40_000, int), [1]])
    if kind == "many shared tiles":
        a = (rng.random(600_000) < 0.33).astype(int)
        a[::5000] += rng.integers(1, 300, 120)
        return np.r_[a, 2_000_000]
    if kind == "most rows of one workgroup":           # and one row more: the second tile, the fourth
        return np.r_[tile, 5, np.zeros(2 * SHARE - 2, int), tile - 5, 1, tile - 1, 5, np.zeros(2 * SHARE - 1, int), tile - 5, 1, 3 * tile]
    if kind == "borders of pieces":                    # at whole and broken flag words, at the end of the tile, several at one position
        a = np.zeros(12 * SHARE, int)
        for i, n in enumerate([128, 127, 129, 0, 1, 31, 32, 33, 96, 0, 7]):
            a[i * SHARE + 5], a[(i + 1) * SHARE - 1], a[(i + 1) * SHARE] = n, 1 + i % 2, 3 * (i % 3)
        return np.r_[np.zeros(SHARE - 77, int), tile // 2, a, 3, np.zeros(3 * SHARE, int), tile // 2, np.zeros(9, int), 40 * SHARE]
    n = {"at the rule": 0, "beyond the rule": 1}[kind]   # three rows per entry, or three rows more
    return np.r_[np.ones(20_000, int), np.zeros(40_000 + 3 * n, int)]


KINDS = ["one row", "one row of many tiles", "starts at tile borders", "empty rows around", "long runs of empty rows",
         "last row of a round", "almost empty rows", "rows of a wave", "some tiles with empty rows", "zipf", "at the rule", "beyond the rule",
         "sorted by degree", "rows of many tiles among empty ones", "many shared tiles", "most rows of one workgroup", "borders of pieces"]


@pytest.mark.parametrize("variant", ["mfma", "shuffle"])
@pytest.mark.parametrize("kind", KINDS)
def test_csr_plan_matches_the_oracle(kind, variant):
    # the tile of a vector depends on its length: two rounds settle it
    tile = 16384
    for _ in range(2):
        lengths = lengths_of(kind, tile)
        nnz = int(lengths.sum())
        tile = B.mmv_tile_elems(B.MMV_OP_SPMV_CSR, B.MMV_F32_F32, nnz)
    n_rows, n_cols = len(lengths), 701
    rowptr = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)
    rng = np.random.default_rng(43)
    col = rng.integers(0, n_cols, nnz, dtype=np.int32)
    val = rng.integers(-3, 4, nnz).astype(np.float32)
    x = rng.integers(-2, 3, n_cols).astype(np.float32)
    want = oracle.spmv_csr(n_rows, n_cols, rowptr, col, val, x)
    d = [dev(a) for a in (rowptr, col, val, x)]
    ws = torch.full((B.mmv_spmv_csr_workspace_bytes(n_rows, nnz),), 0xA5, dtype=torch.uint8, device="cuda")
    y = torch.full((n_rows,), 9.0, device="cuda")
    B.mmv_spmv_csr(n_rows, n_cols, *d, y=y, variant=variant, ws=ws)
    torch.cuda.synchronize()
    assert B.mmv_workspace_status(ws) == 0
    assert np.array_equal(y.cpu().numpy().astype(np.float64), want)
    ws.fill_(0x5A)
    B.mmv_spmv_csr_prepare(n_rows, n_cols, d[0], d[1], ws=ws)
    for _ in range(2):
        y.fill_(5.0)
        B.mmv_spmv_csr_run(n_rows, n_cols, *d, ws=ws, y=y, variant=variant)
        torch.cuda.synchronize()
        assert B.mmv_workspace_status(ws) == 0
        assert np.array_equal(y.cpu().numpy().astype(np.float64), want)
