"""Calls whose launch ahead of the main kernel is gone or shared: a single tile (nothing is zeroed before it), byte flags
(packed in the launch that zeroes, or that counts the segment starts), on workspaces full of garbage."""
import numpy as np
import pytest
import torch

import oracle
from paper_2506_23906_amd import binding as B
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
