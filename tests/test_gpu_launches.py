"""Calls on workspaces full of garbage: short vectors, before whose kernels nothing is zeroed (longer ones: test_gpu_single_pass.py),
and the plans of two-step products, which any other call on their workspace ends."""
import numpy as np
import pytest
import torch

import oracle
from paper_2506_23906_amd import binding as B
from paper_2506_23906_amd import workloads as W
from parity_util import dev, flags_dev

pytestmark = pytest.mark.gpu


def garbage(nbytes):
    return torch.full((max(nbytes, 256),), 0xFF, dtype=torch.uint8, device="cuda")


@pytest.mark.parametrize("packed", [True, False])
@pytest.mark.parametrize("dtype", [np.int8, np.float32])
def test_one_tile_and_more_on_a_workspace_of_garbage(packed, dtype):
    rng = np.random.default_rng(81)
    dt = B.MMV_I8_I32 if dtype == np.int8 else B.MMV_F32_F32
    ff = B.MMV_FLAGS_PACKED32 if packed else B.MMV_FLAGS_U8
    tile = B.mmv_tile_elems(B.MMV_OP_SEGSCAN, dt, 1)
    sum_tile = B.mmv_tile_elems(B.MMV_OP_SEGSUM, dt, 1)
    for n in sorted({1, 33, 1000, tile - 1, tile, tile + 1, 2 * tile + 5, sum_tile, sum_tile + 1, 9 * sum_tile + 31, 70 * sum_tile + 1}):
        x = rng.integers(-3, 4, size=n).astype(dtype)
        for density in (0.0, 0.05, 1.0):
            f = (rng.random(n) < density) * rng.integers(1, 256, size=n)
            f = (f if not packed else f != 0).astype(np.uint8)
            print(packed, dtype.__name__, n, density, flush=True)
            for variant in ("mfma", "shuffle"):
                ws = garbage(B.mmv_workspace_bytes(B.MMV_OP_SEGSCAN, dt, ff, n))
                z = B.mmv_segscan(dev(x), flags_dev(f, packed), n=n, variant=variant, ws=ws)
                assert B.mmv_workspace_status(ws) == 0
                assert np.array_equal(z.cpu().numpy().astype(np.float64), oracle.segscan(x, f).astype(np.float64))
                ws = garbage(B.mmv_workspace_bytes(B.MMV_OP_SEGSUM, dt, ff, n))
                out, nseg = B.mmv_segsum(dev(x), flags_dev(f, packed), n=n, variant=variant, ws=ws)
                assert B.mmv_workspace_status(ws) == 0
                ref = oracle.segsum(x, f)
                assert int(nseg.item()) == len(ref)
                assert np.array_equal(out.cpu().numpy()[:len(ref)].astype(np.float64), ref.astype(np.float64))
                ws = garbage(B.mmv_workspace_bytes(B.MMV_OP_SCAN, dt, ff, n))
                z = B.mmv_scan(dev(x), n=n, variant=variant, ws=ws)
                assert B.mmv_workspace_status(ws) == 0
                assert np.array_equal(z.cpu().numpy().astype(np.float64), oracle.scan(x).astype(np.float64))


def test_calls_go_to_the_current_stream():
    side = torch.cuda.Stream()
    assert B._stream_ptr(None) == int(torch.cuda.current_stream().cuda_stream)
    with torch.cuda.stream(side):
        assert B._stream_ptr(None) == int(side.cuda_stream)
    assert B._stream_ptr(side) == int(side.cuda_stream)


MARK_WORD = 34   # of the workspace header: what mmv_spmv_*_prepare leaves there (0: no plan)


@pytest.mark.parametrize("kind", ["coo", "csr"])
@pytest.mark.parametrize("nnz", [700, 3 * 16384 + 5])          # a product of one tile, and of several
def test_one_tile_calls_end_the_plan_of_a_workspace(kind, nnz):
    n_rows, n_cols, n = 5000, 4000, 1000
    row, col, val, xv = W.spmv_coo_zipf(n_rows, n_cols, nnz, cap=900, seed=5)
    rt, rpt, ct, vt, xt = dev(row), dev(W.csr_rowptr(row, n_rows)), dev(col), dev(val), dev(xv)
    f = np.zeros(n, dtype=np.uint8)
    f[::7] = 1
    x8, x32 = torch.ones(n, dtype=torch.int8, device="cuda"), torch.ones(n, dtype=torch.float32, device="cuda")
    bits, by = flags_dev(f, True), flags_dev(f, False)
    calls = {"scd": (B.MMV_OP_SEGSUM_SCD, lambda ws: B.mmv_segsum_scd(x8, bits, ws=ws)),
             "scd bytes": (B.MMV_OP_SEGSUM_SCD, lambda ws: B.mmv_segsum_scd(x32, by, ws=ws)),
             "sscr": (B.MMV_OP_SEGSCAN_SSCR, lambda ws: B.mmv_segscan_sscr(x32, bits, ws=ws)),
             "segscan": (B.MMV_OP_SEGSCAN, lambda ws: B.mmv_segscan(x32, bits, ws=ws)),
             "segsum": (B.MMV_OP_SEGSUM, lambda ws: B.mmv_segsum(x32, bits, ws=ws)),
             "scan": (B.MMV_OP_SCAN, lambda ws: B.mmv_scan(x8, ws=ws, variant="shuffle"))}
    plan_bytes = (B.mmv_workspace_bytes(B.MMV_OP_SPMV_COO, B.MMV_F32_F32, B.MMV_FLAGS_PACKED32, len(val)) if kind == "coo"
                  else B.mmv_spmv_csr_workspace_bytes(n_rows, len(val)))
    for name, (op, call) in calls.items():
        print(kind, nnz, name, flush=True)
        ws = torch.zeros(max([plan_bytes] + [B.mmv_workspace_bytes(op, dt, ff, n) for dt in (B.MMV_I8_I32, B.MMV_F32_F32)
                                             for ff in (B.MMV_FLAGS_U8, B.MMV_FLAGS_PACKED32)]), dtype=torch.uint8, device="cuda")
        if kind == "coo":
            B.mmv_spmv_coo_prepare(n_rows, n_cols, rt, ct, ws=ws)
        else:
            B.mmv_spmv_csr_prepare(n_rows, n_cols, rpt, ct, ws=ws)
        mark = ws[4 * MARK_WORD:4 * MARK_WORD + 4].view(torch.int32)
        run = ((lambda y: B.mmv_spmv_coo_run(n_rows, n_cols, rt, ct, vt, xt, ws, y=y)) if kind == "coo" else
               (lambda y: B.mmv_spmv_csr_run(n_rows, n_cols, rpt, ct, vt, xt, ws, y=y)))
        y = torch.full((n_rows,), 9.0, device="cuda")
        for _ in range(2):                                     # a run keeps the mark
            run(y)
            assert int(mark.item()) != 0 and B.mmv_workspace_status(ws) == 0
        call(ws)
        assert int(mark.item()) == 0 and B.mmv_workspace_status(ws) == 0      # (before the run that relies on it)
        run(y)
        assert B.mmv_workspace_status(ws) == 2 and bool((y == 0).all())
