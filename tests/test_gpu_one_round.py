"""Scans of 8- and 16-bit values in one round of three workgroups per compute unit: up to 768 tiles of 16384 elements, then tiles of
16384 and of 32768 that make 768 together, up to 25165824 elements; 16-bit values only from 16777217
elements on, mmv_scan of them only without the matrix cores.  Whole numbers: exact."""
import numpy as np
import pytest
import torch

import oracle
from paper_2506_23906_amd import binding as B
from parity_util import dev, flags_dev

pytestmark = pytest.mark.gpu
UNIT, ROUND = 16384, 768
TYPES = {"f16": (np.float16, torch.float16), "bf16": (np.float32, torch.bfloat16), "i8": (np.int8, torch.int8), "u8": (np.uint8, torch.uint8)}


@pytest.mark.parametrize("variant", ["mfma", "shuffle"])
@pytest.mark.parametrize("dt", list(TYPES))
def test_borders_of_the_form(dt, variant):
    rng = np.random.default_rng(2390710)
    if dt in ("f16", "bf16"):
        sizes = [1024 * UNIT, 1024 * UNIT + 1, 1100 * UNIT + 4321, 2 * ROUND * UNIT - 3, 2 * ROUND * UNIT + 1]
    else:
        sizes = [(1 << 22) + 1, ROUND * UNIT - 31, ROUND * UNIT + 1, ROUND * UNIT + 5 * UNIT + 2049, 2 * ROUND * UNIT, 2 * ROUND * UNIT + 1]
    npt, tt = TYPES[dt]
    x = (rng.integers(0, 256, size=max(sizes)) if dt == "u8" else rng.integers(-1, 2, size=max(sizes))).astype(npt)
    for n in sizes:
        xt = dev(x[:n]).to(tt)
        code = B._DTYPES[tt]
        for density in (0.0, 2.0 / UNIT, 0.2):                  # carries through every tile, across some, inside rows
            f = (rng.random(n, dtype=np.float32) < density).astype(np.uint8)
            print(dt, variant, n, density, flush=True)
            packed = n % 2 == 0
            ff = B.MMV_FLAGS_PACKED32 if packed else B.MMV_FLAGS_U8
            ws = torch.full((B.mmv_workspace_bytes(B.MMV_OP_SEGSCAN, code, ff, n),), 0xFF, dtype=torch.uint8, device="cuda")
            z = B.mmv_segscan(xt, flags_dev(f, packed), n=n, variant=variant, ws=ws)
            assert B.mmv_workspace_status(ws) == 0
            assert np.array_equal(z.cpu().numpy().astype(np.float64), oracle.segscan(x[:n], f).astype(np.float64))
        ws = torch.full((B.mmv_workspace_bytes(B.MMV_OP_SCAN, code, B.MMV_FLAGS_PACKED32, n),), 0xFF, dtype=torch.uint8, device="cuda")
        z = B.mmv_scan(xt, n=n, variant=variant, ws=ws)
        assert B.mmv_workspace_status(ws) == 0
        assert np.array_equal(z.cpu().numpy().astype(np.float64), oracle.scan(x[:n]).astype(np.float64))
