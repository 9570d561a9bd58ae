"""Long sums whose kernels look after the end of the vector by the range check of their loads: what lies behind values and flags is
not zero there, and the results end where they should."""
import numpy as np
import pytest
import torch

from paper_2506_23906_amd import binding as B
from parity_util import dev, flags_dev

pytestmark = pytest.mark.gpu
BEHIND = 300_000


def sums(x, f):
    f = f.copy()
    f[0] = 1
    return np.add.reduceat(x.astype(np.int64), np.flatnonzero(f))


def behind(values, n, fill, dtype):
    t = torch.full((n + BEHIND,), fill, dtype=dtype, device="cuda")
    t[:n] = values[:n]
    return t


@pytest.mark.parametrize("variant", ["mfma", "shuffle"])
@pytest.mark.parametrize("dt,base", [(torch.int8, 512 * 4 * 16384), (torch.float16, 512 * 2 * 16384), (torch.float32, 3 << 20), (torch.float32, 512 * 131072)])
def test_sums(dt, base, variant):
    rng = np.random.default_rng(base)
    # in a word, a row, a chunk, behind whole waves
    for ragged in (1, 17, 2047, 16385 + 31) if base < 1 << 24 else (17, 16385 + 31):
        n = base + ragged
        x = rng.integers(-3, 4, size=n).astype(np.int8)
        xt = behind(dev(x).to(dt), n, 5, dt)
        for density in (0.0, 1e-3, 0.3) if base < 1 << 24 else (1e-3,):
            f = (rng.random(n, dtype=np.float32) < density).astype(np.uint8)
            words = (n + 31) // 32
            bits = behind(flags_dev(f, True), words, -1, torch.int32)
            if n % 32:
                bits[words - 1] |= -1 << (n % 32)
            ref = sums(x, f)
            for flags in (bits[:words], behind(dev(f), n, 255, torch.uint8)[:n]):
                out = torch.full((len(ref) + 5000,), 99, dtype=B._OUT_DTYPE[B._DTYPES[dt]], device="cuda")
                _, nseg = B.mmv_segsum(xt[:n], flags, n=n, out=out, variant=variant)
                assert int(nseg.item()) == len(ref), (n, density)
                assert np.array_equal(out[:len(ref)].cpu().numpy().astype(np.int64), ref) and bool((out[len(ref):] == 99).all()), (n, density)


@pytest.mark.parametrize("variant", ["mfma", "shuffle"])
@pytest.mark.parametrize("nnz", [1, 3, 1023, 8 * 1024 + 2, 1_000_003, 5_000_001])
def test_products(nnz, variant):
    """Columns behind the last entry that lie far outside x, next to an x that begins with an infinity."""
    rng = np.random.default_rng(nnz)
    n_rows = max(1, nnz // 7)
    row = np.sort(rng.integers(0, n_rows, size=nnz)).astype(np.int32)
    col = rng.integers(1, 1000, size=nnz).astype(np.int32)
    val, x = rng.integers(-3, 4, size=nnz).astype(np.float32), rng.integers(-3, 4, size=1000).astype(np.float32)
    x[0] = np.inf
    ref = np.bincount(row, weights=val.astype(np.float64) * x[col], minlength=n_rows)
    rowptr = np.searchsorted(row, np.arange(n_rows + 1)).astype(np.int32)
    rt, ct, vt = behind(dev(row), nnz, 0x7FFFFFF0, torch.int32), behind(dev(col), nnz, 0x3FFFFFF0, torch.int32), behind(dev(val), nnz, 7.0, torch.float32)
    y = B.mmv_spmv_coo(n_rows, 1000, rt[:nnz], ct[:nnz], vt[:nnz], dev(x), variant=variant)
    assert np.array_equal(y.cpu().numpy().astype(np.float64), ref)
    y = B.mmv_spmv_csr(n_rows, 1000, dev(rowptr), ct[:nnz], vt[:nnz], dev(x), nnz=nnz, variant=variant)
    assert np.array_equal(y.cpu().numpy().astype(np.float64), ref)
