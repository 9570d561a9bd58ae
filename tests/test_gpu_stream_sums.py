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


def test_sums_of_more_tiles_than_the_tables_without_prefix_sums_cover():
    for dtype, n in ((torch.float32, 4100 * 128 * UNIT + 777), (torch.int8, 4200 * 131072 + 5)):
        print("long sum", dtype, n, flush=True)
        length = 1000
        f = torch.zeros(n, dtype=torch.uint8, device="cuda")
        f[::length] = 1
        x = torch.full((n,), 2, dtype=dtype, device="cuda")
        count = (n + length - 1) // length
        out, nseg = B.mmv_segsum(x, f, n=n, out=torch.empty(count, dtype=torch.int32 if dtype == torch.int8 else dtype, device="cuda"))
        assert int(nseg.item()) == count
        assert bool((out[:-1] == 2 * length).all()) and float(out[-1]) == 2 * (n - (count - 1) * length)
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


def test_csr_of_more_tiles_than_the_tables_without_prefix_sums_cover():
    length, n_cols = 1000, 4096
    n_rows = 4100 * 128 * UNIT // length + 3
    nnz = n_rows * length
    rowptr = torch.arange(0, nnz + 1, length, dtype=torch.int32, device="cuda")
    col = (torch.arange(nnz, dtype=torch.int32, device="cuda") % n_cols)
    val = torch.ones(nnz, dtype=torch.float32, device="cuda")
    x = torch.full((n_cols,), 2.0, device="cuda")
    print("long csr", nnz, flush=True)
    y = B.mmv_spmv_csr(n_rows, n_cols, rowptr, col, val, x)
    assert bool((y == 2.0 * length).all())


@pytest.mark.parametrize("variant", ["mfma", "shuffle"])
def test_borders_of_the_form_for_short_vectors(variant):
    """256 tiles of 8 to 16 units, 512 (sums) of 8 to 16, 768 (sums without the matrix cores) of up to 16, and what lies
    just beyond each; ragged ends in the first and in the second unit of a wave."""
    rng = np.random.default_rng(74)
    for n in [2 * UNIT + 3, 9 * UNIT + 5, 15 * UNIT - 1, 256 * 8 * UNIT, 256 * 8 * UNIT + 1, 256 * 11 * UNIT + 31, 256 * 16 * UNIT, 256 * 16 * UNIT + 1,
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
