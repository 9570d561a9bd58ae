"""COMPRESS where its waves compact pieces of 1024 positions through LDS: borders of pieces, groups and tiles, byte masks
that the kernel reads itself, output offsets and capacities that are no multiple of four, densities around the
border between the two paths of a wave (1 selected position in 32)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2506_23906_amd import binding as B
from parity_util import dev, flags_dev

pytestmark = pytest.mark.gpu


def check(n, m, x, packed, capacity):
    print("compress", n, int((m != 0).sum()), packed, capacity, flush=True)
    ref = oracle.compress(x, m) if x is not None else np.flatnonzero(m).astype(np.int32)
    out = torch.full((max(capacity, 1) + 9,), -7, dtype=torch.int32, device="cuda")
    ws = B.new_workspace(B.MMV_OP_COMPRESS, B.MMV_I8_I32, B._flag_fmt(flags_dev(m, packed)), n)
    _, count = B.mmv_compress(None if x is None else dev(x), flags_dev(m, packed), n, out=out[:capacity], ws=ws)
    assert B.mmv_workspace_status(ws) == 0
    got = out.cpu().numpy()
    k = min(capacity, len(ref))
    assert int(count.item()) == len(ref)
    assert np.array_equal(got[:k], ref[:k])
    assert (got[k:] == -7).all()


@pytest.mark.parametrize("packed", [True, False])
def test_pieces(packed):
    rng = np.random.default_rng(91)
    for n in (1023, 1024, 1025, 8191, 8192 + 1, (1 << 22) - 3, (1 << 22) + 1, (1 << 22) + 64 * 4096 + 1027):
        for density in (0.02, 0.03125, 0.05, 0.3, 0.97, 1.0):
            m = (rng.random(n) < density) * rng.integers(1, 256, size=n)
            m = (m if not packed else m != 0).astype(np.uint8)
            x = rng.integers(-2**31, 2**31, size=n, dtype=np.int64).astype(np.int32)
            count = int((m != 0).sum())
            for capacity in (n, max(1, count - 1), max(1, count // 2 + 1)):
                check(n, m, x if capacity != n or density != 0.3 else None, packed, capacity)


@pytest.mark.parametrize("packed,n", [(True, (1 << 26) + 1027), (False, (1 << 26) + 5), (True, (1 << 27) + 77), (False, (1 << 28) + 3)])
def test_long_masks_dense_and_sparse_stretches(packed, n):
    rng = np.random.default_rng(92)
    m = np.zeros(n, dtype=np.uint8)
    edges = [0, n // 5, n // 5 + 3 * 65536, n // 2, n]
    for (a, b), density in zip(zip(edges[:-1], edges[1:]), (0.3, 0.0005, 0.04, 0.01)):
        for c in range(a, b, 1 << 25):
            d = min(b, c + (1 << 25))
            m[c:d] = rng.random(d - c, dtype=np.float32) < density
    x = np.arange(n, dtype=np.uint32).view(np.int32) * np.int32(-1640531527)
    check(n, m, x, packed, int(m.sum()))


@pytest.mark.parametrize("packed", [True, False])
@pytest.mark.parametrize("base", [1 << 18, 1 << 22, 1 << 26])            # 16 words per wave in one launch; 64; two groups of them
def test_set_bits_behind_the_mask_do_not_count(base, packed):
    """Ragged ends of words, of lanes, of waves that have no positions; what lies behind mask and values is all ones."""
    rng = np.random.default_rng(base)
    for ragged in (1, 15, 31, 33, 64, 1025, 40_001):
        n = base + ragged
        m = (rng.random(n, dtype=np.float32) < 0.1).astype(np.uint8)
        x = rng.integers(-2 ** 31, 2 ** 31, size=n, dtype=np.int64).astype(np.int32)
        xt = torch.full((n + 70_000,), -1, dtype=torch.int32, device="cuda")
        xt[:n] = dev(x)
        if packed:
            words = (n + 31) // 32
            mask = torch.full((words + 4000,), -1, dtype=torch.int32, device="cuda")
            mask[:words] = flags_dev(m, True)[:words]
            if n % 32:
                mask[words - 1] |= -1 << (n % 32)
            mask = mask[:words]
        else:
            mask = torch.full((n + 70_000,), 255, dtype=torch.uint8, device="cuda")
            mask[:n] = dev(m)
            mask = mask[:n]
        ref = x[m == 1]
        out = torch.full((len(ref) + 70_000,), 7, dtype=torch.int32, device="cuda")
        _, count = B.mmv_compress(xt[:n], mask, n, out=out)
        assert int(count.item()) == len(ref), (packed, n)
        assert np.array_equal(out[:len(ref)].cpu().numpy(), ref) and bool((out[len(ref):] == 7).all()), (packed, n)
