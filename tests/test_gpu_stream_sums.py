"""The segmented sum of fp32 values and SpMV where their kernel can go wrong: borders of rows, units of 1024 elements and
tiles of 8 to 128 units, the two ways of counting the segment starts inside a tile (up to 16 units, more), tiles that no
longer fit the tables without prefix sums, a vector x with more entries than 32-bit byte offsets reach, a ragged end in
front of an infinite x[0].  Values are small integers, so that every order of additions gives the same fp32 result."""
import numpy as np
import pytest
import torch

import oracle
from paper_2506_23906_amd import binding as B
from paper_2506_23906_amd import workloads as W
from parity_util import dev, flags_dev

pytestmark = pytest.mark.gpu
UNIT = 1024


def segment_patterns(n, rng):
    some = (rng.random(n) < 0.02).astype(np.uint8)
    many = (rng.random(n) < 0.4).astype(np.uint8)
    at_units = np.zeros(n, dtype=np.uint8)
    at_units[::UNIT] = 1
    before_units = np.zeros(n, dtype=np.uint8)
    before_units[UNIT - 1::UNIT] = 1
    last = np.zeros(n, dtype=np.uint8)
    last[-1] = 1
    return [("none", np.zeros(n, dtype=np.uint8)), ("all", np.ones(n, dtype=np.uint8)), ("some", some), ("many", many),
            ("unit starts", at_units), ("before unit starts", before_units), ("last", last)]


@pytest.mark.parametrize("variant", ["mfma", "shuffle"])
def test_sums_at_borders(variant):
    rng = np.random.default_rng(71)
    # 8 units per tile; 8 and 16 units of a round of 512 or 768 tiles; more than 16
    sizes = [1, 31, 32, 33, UNIT - 1, UNIT, UNIT + 1, 8 * UNIT - 1, 8 * UNIT, 8 * UNIT + 1, 20 * UNIT + 77,
             512 * 8 * UNIT + 1, 768 * 8 * UNIT + 1, 512 * 16 * UNIT, 512 * 16 * UNIT + 1, 768 * 16 * UNIT + 33, 768 * 17 * UNIT + 5]
    for n in sizes:
        x = rng.integers(-3, 4, size=n).astype(np.float32)
        xt = dev(x)
        for name, f in segment_patterns(n, rng) if n < 30 * UNIT else segment_patterns(n, rng)[2:4]:
            print("sum", variant, n, name, flush=True)
            ref = oracle.segsum(x, f)
            for capacity in (len(ref), max(1, len(ref) // 2)):
                out = torch.full((len(ref) + 3,), 99.0, dtype=torch.float32, device="cuda")
                ws = B.new_workspace(B.MMV_OP_SEGSUM, B.MMV_F32_F32, B.MMV_FLAGS_PACKED32, n)
                _, nseg = B.mmv_segsum(xt, flags_dev(f, True), n=n, out=out[:capacity], variant=variant, ws=ws)
                assert B.mmv_workspace_status(ws) == 0
                got = out.cpu().numpy()
                assert int(nseg.item()) == len(ref)
                assert np.array_equal(got[:capacity].astype(np.float64), ref[:capacity])
                assert (got[capacity:] == 99.0).all()


def varied_lengths(total, shortest):
    """Lengths of shortest .. shortest + 600 that follow no period of a tile, about `total` together."""
    k = torch.arange(int(total // (shortest + 300)) + 1, device="cuda")
    return shortest + (k * 389) % 601


def test_sums_of_more_tiles_than_the_tables_without_prefix_sums_cover():
    for dtype, total in ((torch.float32, 4110 * 128 * UNIT + 777), (torch.int8, 4300 * 131072 + 5)):
        lengths = varied_lengths(total, 700)
        count, n = lengths.numel(), int(lengths.sum())
        assert n > (4097 * 128 * UNIT if dtype == torch.float32 else 4200 * 131072)
        print("long sum", dtype, n, flush=True)
        f = torch.zeros(n, dtype=torch.uint8, device="cuda")
        f[torch.cumsum(lengths, 0) - lengths] = 1
        value = torch.arange(count, device="cuda") % 7 - 3          # of every element of a segment
        x = value.to(dtype).repeat_interleave(lengths)
        odt = torch.int32 if dtype == torch.int8 else dtype
        out, nseg = B.mmv_segsum(x, f, n=n, out=torch.full((count + 5,), 99, dtype=odt, device="cuda"))
        assert int(nseg.item()) == count
        assert torch.equal(out[:count].long(), value * lengths) and bool((out[count:] == 99).all())
        del f, x, out


@pytest.mark.parametrize("variant", ["mfma", "shuffle"])
def test_spmv_at_borders(variant):
    rng = np.random.default_rng(72)
    for nnz in [1, 33, UNIT - 1, UNIT, UNIT + 1, 8 * UNIT, 8 * UNIT + 1, 37 * UNIT + 5, 768 * 8 * UNIT + 3, 768 * 17 * UNIT + 1]:
        for mean in (1.5, 300.0):
            n_rows = max(2, int(nnz / mean))
            row = np.sort(rng.integers(0, n_rows, size=nnz)).astype(np.int32)      # some rows empty
            if mean > 2:
                row = (row // 2) if nnz % 2 else np.sort(np.concatenate([row[: nnz - n_rows], np.arange(n_rows, dtype=np.int32)]) if nnz > n_rows else row)
            n_cols = 5000
            col = rng.integers(1, n_cols, size=nnz, dtype=np.int32)
            val = rng.integers(-2, 3, size=nnz).astype(np.float32)
            x = rng.integers(-2, 3, size=n_cols).astype(np.float32)
            x[0] = np.inf                                                          # no entry refers to it
            ref = np.zeros(n_rows)
            np.add.at(ref, row, val.astype(np.float64) * x[col])
            rowptr = W.csr_rowptr(row, n_rows)
            args = [dev(a) for a in (col, val, x)]
            print("spmv", variant, nnz, n_rows, flush=True)
            y = B.mmv_spmv_coo(n_rows, n_cols, dev(row), *args, variant=variant)
            assert np.array_equal(y.cpu().numpy().astype(np.float64), ref)
            y = B.mmv_spmv_csr(n_rows, n_cols, dev(rowptr), *args, variant=variant)
            assert np.array_equal(y.cpu().numpy().astype(np.float64), ref)
            ws = B.mmv_spmv_csr_prepare(n_rows, n_cols, dev(rowptr), args[0])
            for _ in range(2):
                y = B.mmv_spmv_csr_run(n_rows, n_cols, dev(rowptr), *args, ws, variant=variant)
                assert np.array_equal(y.cpu().numpy().astype(np.float64), ref)


def test_spmv_with_columns_beyond_32_bit_byte_offsets():
    n_cols, nnz, n_rows = (1 << 30) + 1000, 40_000, 500
    rng = np.random.default_rng(73)
    row = np.sort(rng.integers(0, n_rows, size=nnz)).astype(np.int32)
    col = np.where(rng.random(nnz) < 0.5, rng.integers(0, 1000, size=nnz), n_cols - 1 - rng.integers(0, 900, size=nnz)).astype(np.int32)
    val = rng.integers(-2, 3, size=nnz).astype(np.float32)
    x = torch.zeros(n_cols, dtype=torch.float32, device="cuda")
    x[:1000] = 1.0
    x[-1000:] = 3.0
    xc = np.where(col < 1000, 1.0, 3.0)
    ref = np.zeros(n_rows)
    np.add.at(ref, row, val * xc)
    for variant in ("mfma", "shuffle"):
        y = B.mmv_spmv_coo(n_rows, n_cols, dev(row), dev(col), dev(val), x, variant=variant)
        assert np.array_equal(y.cpu().numpy().astype(np.float64), ref)
        y = B.mmv_spmv_csr(n_rows, n_cols, dev(W.csr_rowptr(row, n_rows)), dev(col), dev(val), x, variant=variant)
        assert np.array_equal(y.cpu().numpy().astype(np.float64), ref)


@pytest.mark.parametrize("nnz", [40_001, 4_300_001])                 # a tile that a wave loads at once; the form that gathers by buffer loads
@pytest.mark.parametrize("more", [-1, 0, 1, 1000])
def test_spmv_at_the_reach_of_32_bit_byte_offsets(more, nnz):
    """x of 2^30 + more entries, of which the last and the first are used; behind the last entry lie columns far outside x."""
    n_cols, n_rows = (1 << 30) + more, nnz // 7
    rng = np.random.default_rng(nnz + more)
    row = np.sort(rng.integers(0, n_rows, size=nnz)).astype(np.int32)
    places = np.array([0, 1, n_cols - 2, n_cols - 1])
    which = rng.integers(0, 4, size=nnz)
    val = rng.integers(-2, 3, size=nnz).astype(np.float32)
    x = torch.zeros(n_cols, dtype=torch.float32, device="cuda")
    x[places.tolist()] = torch.tensor([1.0, 3.0, 5.0, 7.0], device="cuda")
    ref = np.bincount(row, weights=val.astype(np.float64) * np.array([1.0, 3.0, 5.0, 7.0])[which], minlength=n_rows)
    col = torch.full((nnz + 64,), 0x7FFFFFF0, dtype=torch.int32, device="cuda")
    col[:nnz] = dev(places[which].astype(np.int32))
    rowptr = dev(np.searchsorted(row, np.arange(n_rows + 1)).astype(np.int32))
    for variant in ("mfma", "shuffle"):
        y = B.mmv_spmv_coo(n_rows, n_cols, dev(row), col[:nnz], dev(val), x, variant=variant)
        assert np.array_equal(y.cpu().numpy().astype(np.float64), ref), variant
        y = B.mmv_spmv_csr(n_rows, n_cols, rowptr, col[:nnz], dev(val), x, variant=variant)
        assert np.array_equal(y.cpu().numpy().astype(np.float64), ref), variant


def test_csr_of_more_tiles_than_the_tables_without_prefix_sums_cover():
    n_cols = 4096
    lengths = varied_lengths(1.5 * 4110 * 128 * UNIT, 700)
    lengths[1::3] = 0                                                # a third of the rows is empty
    n_rows, nnz = lengths.numel(), int(lengths.sum())
    assert 4097 * 128 * UNIT < nnz < 2 ** 31
    rowptr = torch.zeros(n_rows + 1, dtype=torch.int32, device="cuda")
    rowptr[1:] = torch.cumsum(lengths, 0).int()
    col = (torch.arange(nnz, dtype=torch.int32, device="cuda") % n_cols)
    value = torch.arange(n_rows, device="cuda") % 5 - 2              # of every entry of a row
    val = value.float().repeat_interleave(lengths)
    x = torch.full((n_cols,), 2.0, device="cuda")
    print("long csr", nnz, flush=True)
    y = B.mmv_spmv_csr(n_rows, n_cols, rowptr, col, val, x, y=torch.full((n_rows,), 77.0, device="cuda"))
    assert torch.equal(y.long(), 2 * value * lengths)
    ws = B.mmv_spmv_csr_prepare(n_rows, n_cols, rowptr, col)
    y = B.mmv_spmv_csr_run(n_rows, n_cols, rowptr, col, val, x, ws, y=torch.full((n_rows,), 77.0, device="cuda"), variant="shuffle")
    assert torch.equal(y.long(), 2 * value * lengths)


@pytest.mark.parametrize("variant", ["mfma", "shuffle"])
def test_borders_of_the_form_for_short_vectors(variant):
    """256 tiles of 8 to 16 units, 512 (sums) of 8 to 16, 768 (sums without the matrix cores) of up to 16, and what lies
    just beyond each; ragged ends in the first and in the second unit of a wave."""
    rng = np.random.default_rng(74)
    for n in [2 * UNIT + 3, 9 * UNIT + 5, 15 * UNIT - 1, 256 * 8 * UNIT, 256 * 8 * UNIT + 1, 256 * 11 * UNIT + 31, 3 * 1024 * UNIT + 1, 256 * 13 * UNIT + 31, 256 * 16 * UNIT, 256 * 16 * UNIT + 1,
              512 * 12 * UNIT + 7, 512 * 16 * UNIT + 1, 768 * 16 * UNIT, 768 * 16 * UNIT + 1]:
        x = rng.integers(-3, 4, size=n).astype(np.float32)
        for density in (0.0002, 0.3):
            f = (rng.random(n) < density).astype(np.uint8)
            print("short sum", variant, n, density, flush=True)
            ref = oracle.segsum(x, f)
            out, nseg = B.mmv_segsum(dev(x), flags_dev(f, density < 0.1), n=n, out=torch.full((len(ref) + 3,), 99.0, device="cuda"), variant=variant)
            assert int(nseg.item()) == len(ref)
            got = out.cpu().numpy()
            assert np.array_equal(got[:len(ref)].astype(np.float64), ref) and (got[len(ref):] == 99.0).all()
    for nnz in [2 * UNIT + 3, 9 * UNIT + 5, 256 * 8 * UNIT, 256 * 8 * UNIT + 1, 256 * 16 * UNIT, 256 * 16 * UNIT + 1]:
        n_cols, n_rows = 3000, max(2, nnz // 37)
        row = np.sort(rng.integers(0, n_rows, size=nnz)).astype(np.int32)
        col = rng.integers(0, n_cols, size=nnz, dtype=np.int32)
        val, x = rng.integers(-2, 3, size=nnz).astype(np.float32), rng.integers(-2, 3, size=n_cols).astype(np.float32)
        ref = np.bincount(row, weights=val.astype(np.float64) * x[col], minlength=n_rows)
        args = [dev(a) for a in (col, val, x)]
        rowptr = dev(W.csr_rowptr(row, n_rows))
        print("short spmv", variant, nnz, flush=True)
        assert np.array_equal(B.mmv_spmv_coo(n_rows, n_cols, dev(row), *args, variant=variant).cpu().numpy().astype(np.float64), ref)
        assert np.array_equal(B.mmv_spmv_csr(n_rows, n_cols, rowptr, *args, variant=variant).cpu().numpy().astype(np.float64), ref)
        ws = B.mmv_spmv_csr_prepare(n_rows, n_cols, rowptr, args[0])
        assert np.array_equal(B.mmv_spmv_csr_run(n_rows, n_cols, rowptr, *args, ws, variant=variant).cpu().numpy().astype(np.float64), ref)


@pytest.mark.parametrize("variant", ["mfma", "shuffle"])
# products in the form for short vectors and short sums, sums in that form, the form for long vectors
@pytest.mark.parametrize("n", [9 * 8 * UNIT + 700, (3 << 20) + 700, 768 * 17 * UNIT + 900])
def test_non_finite_values_reach_their_own_segment_and_those_of_their_row_of_32(variant, n):
    """Sums and products: a segment that holds an infinity or a NaN has a sum that is not finite, one that lies
    partly in the same (32-aligned) row may have, every other sum is as accurate as without them (within 2e-5 of the sum of
    the magnitudes, the margin of parity_util)."""
    rng = np.random.default_rng(75)
    x = (rng.random(n, dtype=np.float32) * 2 - 1).astype(np.float32)
    f = (rng.random(n) < 0.02).astype(np.uint8)
    quiet = slice(20 * UNIT, 45 * UNIT)                               # units and tiles that lie inside one segment
    f[quiet] = 0
    f[0] = 1
    bad = {5: np.inf, 3 * UNIT - 1: -np.inf, 3 * UNIT + 40: np.nan, 8 * UNIT: np.inf, 16 * UNIT - 1: np.inf, 30 * UNIT + 17: np.inf,
           n - 1: -np.inf, n - 2000: np.nan, n // 2: np.inf}
    f[[8 * UNIT, n // 2 + 1]] = 1                                     # one on a segment start, one right ahead of one
    for p, v in bad.items():
        x[p] = v
    segment = np.cumsum(f) - 1
    starts = np.flatnonzero(f)
    own = np.unique(segment[list(bad)])
    near = np.unique(np.concatenate([segment[p // 32 * 32:p // 32 * 32 + 32] for p in bad]))
    clean = np.ones(len(starts), dtype=bool)
    clean[near] = False
    finite = np.where(np.isfinite(x), x, 0).astype(np.float64)
    ref, size = np.add.reduceat(finite, starts), np.add.reduceat(np.abs(finite), starts)

    def check(got, what):
        print("non-finite", what, variant, n, flush=True)
        assert not np.isfinite(got[own]).any()
        assert (np.abs(got.astype(np.float64) - ref)[clean] <= 2e-5 * np.maximum(size, 1)[clean]).all()

    out, nseg = B.mmv_segsum(dev(x), flags_dev(f, True), n=n, variant=variant)
    assert int(nseg.item()) == len(starts)
    check(out.cpu().numpy()[:len(starts)], "sum")
    # products: one column per entry holds the values, the entries are ones, the rows the segments
    row, col = segment.astype(np.int32), rng.permutation(n).astype(np.int32)
    xv = np.empty(n, dtype=np.float32)
    xv[col] = x
    args = [dev(a) for a in (col, np.ones(n, dtype=np.float32), xv)]
    check(B.mmv_spmv_coo(len(starts), n, dev(row), *args, variant=variant).cpu().numpy(), "coo")
    check(B.mmv_spmv_csr(len(starts), n, dev(W.csr_rowptr(row, len(starts))), *args, variant=variant).cpu().numpy(), "csr")
