"""Scans and sums of short vectors: one launch (the sum carried into a tile comes from the input itself) up to 320 KB of
values and flags, two (from the aggregates of the tiles before) up to 2^21 elements (fp32 sums and 16-bit mmv_scan 3 * 2^20, other mmv_scan 2^22), the single-pass kernels beyond.  Tiles have 2048 elements, a thread takes eight, a wave 512; whole numbers, so results are exact."""
import numpy as np
import pytest
import torch

import oracle
from paper_2506_23906_amd import binding as B
from parity_util import check_scan, check_sum, dev, flags_dev, run_segscan, run_segsum

pytestmark = pytest.mark.gpu
TILE = 2048
TYPES = {"f32": (torch.float32, B.MMV_F32_F32), "f16": (torch.float16, B.MMV_F16_F32), "bf16": (torch.bfloat16, B.MMV_BF16_F32),
         "i8": (torch.int8, B.MMV_I8_I32), "u8": (torch.uint8, B.MMV_U8_XOR)}


MANY_BITS, MANY_BYTES = {4: 288, 2: 240, 1: 96}, {4: 160, 2: 128, 1: 80}      # KB, by the size of a value


def one_launch(dt, flag_bytes):
    """Most elements that one launch takes (8 * flag_bytes: bits of flags per element)."""
    size = torch.empty(0, dtype=TYPES[dt][0]).element_size()
    return int((320 << 10) / (size + flag_bytes)) // 32 * 32


def values(rng, n, dt):
    x = rng.integers(0, 256, size=n) if dt == "u8" else rng.integers(-3, 4, size=n)
    return x.astype({"f32": np.float32, "f16": np.float16, "bf16": np.float32, "i8": np.int8, "u8": np.uint8}[dt])


def garbage(nbytes):
    return torch.full((max(nbytes, 256),), 0xFF, dtype=torch.uint8, device="cuda")


def check(dt, n, packed, f, rng, variant="mfma", scan_too=True):
    x = values(rng, n, dt)
    tt, code = TYPES[dt]
    xt, ft = dev(x).to(tt), flags_dev(f, packed)
    ff = B.MMV_FLAGS_PACKED32 if packed else B.MMV_FLAGS_U8
    ws = garbage(B.mmv_workspace_bytes(B.MMV_OP_SEGSCAN, code, ff, n))
    z = B.mmv_segscan(xt, ft, n=n, variant=variant, ws=ws)
    assert B.mmv_workspace_status(ws) == 0
    assert np.array_equal(z.cpu().numpy().astype(np.float64), oracle.segscan(x, f).astype(np.float64))
    ws = garbage(B.mmv_workspace_bytes(B.MMV_OP_SEGSUM, code, ff, n))
    ref = oracle.segsum(x, f)
    cap = len(ref) - len(ref) // 3                              # an output array that is too short
    out = torch.full((cap + 64,), -77, dtype=B._OUT_DTYPE[code], device="cuda")
    _, nseg = B.mmv_segsum(xt, ft, n=n, out=out[:cap], variant=variant, ws=ws)
    assert B.mmv_workspace_status(ws) == 0 and int(nseg.item()) == len(ref)
    assert np.array_equal(out.cpu().numpy()[:cap].astype(np.float64), ref[:cap].astype(np.float64))
    assert bool((out[cap:] == -77).all())
    if scan_too:
        ws = garbage(B.mmv_workspace_bytes(B.MMV_OP_SCAN, code, ff, n))
        z = B.mmv_scan(xt, n=n, variant=variant, ws=ws)
        assert B.mmv_workspace_status(ws) == 0
        assert np.array_equal(z.cpu().numpy().astype(np.float64), oracle.scan(x).astype(np.float64))


@pytest.mark.parametrize("packed", [True, False])
@pytest.mark.parametrize("dt", list(TYPES))
def test_edges_of_threads_waves_tiles_and_of_the_two_forms(dt, packed):
    rng = np.random.default_rng(2390700)
    line = one_launch(dt, 1 / 8 if packed else 1)
    sizes = [1, 2, 7, 8, 9, 31, 33, 511, 513, TILE - 1, TILE, TILE + 1, 5 * TILE + 511, line - 1, line, line + 1, line + TILE + 9,
             3 << 19, (3 << 19) + 1, (1 << 21) - 5, 1 << 21, (1 << 21) + 1, 3 << 20, (3 << 20) + 1, (1 << 22) - 3, 1 << 22, (1 << 22) + 1]
    for n in sizes:
        for density in (0.0, 3 / n, 0.01, 1.0):
            f = ((rng.random(n) < density) * rng.integers(1, 256, size=n)).astype(np.uint8)
            print(dt, packed, n, density, flush=True)
            check(dt, n, packed, f if not packed else (f != 0).astype(np.uint8), rng)


@pytest.mark.parametrize("n", [9 * TILE + 77, 150 * TILE + 77])          # one launch, two
@pytest.mark.parametrize("packed", [True, False])
def test_single_flags_at_borders(n, packed):
    """One flag per vector, at and around the borders of threads, 128-bit words, waves and tiles, and in the first and last
    positions: what every later tile adds up begins there."""
    rng = np.random.default_rng(2390701)
    at = {0, 1, n - 1, n - 2}
    for b in (8, 16, 128, 512, TILE, 2 * TILE, 3 * TILE + 512, n - n % TILE):
        at |= {b - 1, b, b + 1}
    for p in sorted(at):
        f = np.zeros(n, dtype=np.uint8)
        f[p] = 1
        for dt in ("f32", "f16", "i8") if p % 2 else ("bf16", "u8"):
            print(n, packed, p, dt, flush=True)
            check(dt, n, packed, f, rng, variant="shuffle", scan_too=p == 0)


@pytest.mark.parametrize("n", [60_001, 200_003])
def test_in_place_and_overlapping(n):
    """fp32 results over their own input: never in one launch, where other workgroups still read it."""
    rng = np.random.default_rng(2390702)
    x = values(rng, n, "f32")
    f = (rng.random(n) < 0.001).astype(np.uint8)
    for packed in (True, False):
        for _ in range(3):
            xt = dev(x)
            B.mmv_segscan(xt, flags_dev(f, packed), n=n, z=xt)
            assert np.array_equal(xt.cpu().numpy(), oracle.segscan(x, f).astype(np.float32))
    for _ in range(3):
        xt = dev(x)
        B.mmv_scan(xt, n=n, z=xt)
        assert np.array_equal(xt.cpu().numpy(), oracle.scan(x).astype(np.float32))


@pytest.mark.parametrize("n", [70_000, (1 << 21) - 1, (1 << 22) + 3])    # one launch, two, the single-pass kernels
@pytest.mark.parametrize("variant", ["mfma", "shuffle"])
def test_real_values_starts_and_non_finite_ones(n, variant):
    rng = np.random.default_rng(2390703)
    x = (rng.random(n, dtype=np.float32) * 2 - 1).astype(np.float32)
    f = (rng.random(n) < 0.02).astype(np.uint8)
    check_scan(run_segscan(x, f, variant), x, f)
    out, nseg = run_segsum(x, f, variant)
    check_sum(out, nseg, x, f)
    bad = {5 * 32 + 7: np.inf, 700 * 32 + 11: -np.inf, n - 2048 - 40: np.nan, 0: -0.0}
    for p, v in bad.items():
        x[p] = v
        f[p // 32 * 32 + 32] = 1                                  # the next row of 32 starts a segment
    z = run_segscan(x, f, variant)
    starts = np.flatnonzero(f)
    assert np.array_equal(z[starts].view(np.uint32), x[starts].view(np.uint32))
    with np.errstate(invalid="ignore"):
        ref = oracle.segscan(x, f)
    rows = {p // 32 for p in bad}
    assert set((np.flatnonzero(~np.isfinite(z)) // 32).tolist()) <= rows
    assert not np.isfinite(z[[p for p in bad if p]]).any()        # (an infinity or a NaN: the row scans subtract prefixes)
    if n <= 1 << 21:                                              # no speculation: exactly the values of the definition
        assert np.array_equal(np.isfinite(z), np.isfinite(ref))
        for p in bad:
            assert np.array_equal(z[p:p + 1], ref[p:p + 1].astype(np.float32), equal_nan=True)


def test_graph_replays_and_a_workspace_shared_by_lengths():
    """One workspace, sized for the longest of them, serves vectors of all three forms in turn, also in a graph."""
    rng = np.random.default_rng(2390704)
    sizes = [(1 << 22) + 5, 30_000, 1 << 21, 1, 1_000_000]
    data = []
    ws = garbage(B.mmv_workspace_bytes(B.MMV_OP_SEGSUM, B.MMV_I8_I32, B.MMV_FLAGS_PACKED32, max(sizes)))
    for n in sizes:
        x, f = values(rng, n, "i8"), (rng.random(n) < 0.003).astype(np.uint8)
        assert B.mmv_workspace_bytes(B.MMV_OP_SEGSUM, B.MMV_I8_I32, B.MMV_FLAGS_PACKED32, n) <= ws.numel()
        data.append((dev(x), flags_dev(f, True), n, torch.zeros(n, dtype=torch.int32, device="cuda"),
                     torch.zeros(1, dtype=torch.int64, device="cuda"), oracle.segsum(x, f)))
    g = torch.cuda.CUDAGraph()

    def calls():
        for xt, ft, n, out, nseg, _ in data:
            B.mmv_segsum(xt, ft, n=n, out=out, nseg=nseg, ws=ws)
    calls()
    torch.cuda.synchronize()
    with torch.cuda.graph(g):
        calls()
    for rep in range(4):
        for d in data:
            d[3].zero_(), d[4].zero_()
        if rep:
            torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        for _, _, n, out, nseg, ref in data:
            assert int(nseg.item()) == len(ref) and np.array_equal(out.cpu().numpy()[:len(ref)], ref), (rep, n)


def test_sscr_counts_position_zero_whatever_its_flag():
    """The composition scans flag bytes with element 0 counted as 1, through both forms of a short scan."""
    rng = np.random.default_rng(2390705)
    for n in (100, 250_000, 400_000):
        x, f = values(rng, n, "i8"), (rng.random(n) < 0.01).astype(np.uint8)
        f[0] = 0
        z = B.mmv_segscan_sscr(dev(x), flags_dev(f, True), n=n)
        torch.cuda.synchronize()
        assert np.array_equal(z.cpu().numpy(), oracle.segscan(x, f))


@pytest.mark.parametrize("packed", [True, False])
def test_compress_in_one_launch(packed):
    """Masks of at most 2^21 bits or 2^17 bytes: every workgroup of 8192 positions counts the set bits before its tile itself."""
    rng = np.random.default_rng(2390706)
    line = 1 << (21 if packed else 17)
    for n in (1, 127, 128, 129, 8191, 8192, 8193, 5 * 8192 + 1023, line - 33, line, line + 1):
        for density in (0.0, 2 / n, 0.01, 0.3, 1.0):
            m = (rng.random(n) < density) * rng.integers(1, 256, size=n)
            m = (m if not packed else m != 0).astype(np.uint8)
            x = rng.integers(-2**31, 2**31, size=n, dtype=np.int64).astype(np.int32)
            print(packed, n, density, flush=True)
            ref, pos = oracle.compress(x, m), np.flatnonzero(m).astype(np.int32)
            cap = len(ref) - len(ref) // 3
            for src, want in ((dev(x), ref), (None, pos)):
                out = torch.full((cap + 9,), -7, dtype=torch.int32, device="cuda")
                ws = garbage(B.mmv_workspace_bytes(B.MMV_OP_COMPRESS, B.MMV_I8_I32, B.MMV_FLAGS_PACKED32 if packed else B.MMV_FLAGS_U8, n))
                _, count = B.mmv_compress(src, flags_dev(m, packed), n, out=out[:cap], ws=ws)
                assert B.mmv_workspace_status(ws) == 0 and int(count.item()) == len(want)
                assert np.array_equal(out.cpu().numpy()[:cap], want[:cap]) and bool((out[cap:] == -7).all())


@pytest.mark.parametrize("n", [30_003, 200_003])                       # one launch, two
@pytest.mark.parametrize("dt,big,small", [("f32", 2.0 ** 40, 1.0), ("bf16", 2.0 ** 40, 1.0), ("f16", 2.0 ** 15, 2.0 ** -10), ("f32", 2e38, 0.0)])
def test_sums_across_tiles_are_carried_in_64_bits(n, dt, big, small):
    """big, small, -big, small over and over: in 64 bits every running sum is exact (sums of 2^40 and up to 10^5 ones, of 2^15
    and 10^5 / 2^10; those of whole tiles, which two launches keep in 32 bits, are 1024 smalls), so results are the definition's
    rounded once.  In 32 bits the smalls are lost beside big.  With 2e38 and nothing between, every running sum is 0 or 2e38,
    while two of the same sign overflow 32 bits.  One segment, then one that begins inside a 128-bit word."""
    x = np.tile(np.array([big, small, -big, small] if small else [big, -big, big, -big]), n // 4 + 1)[:n].astype(np.float32)
    xt = dev(x).to(TYPES[dt][0])
    x = xt.float().cpu().numpy()                                       # (as the type holds them)
    for starts in ([], [4 * 777]):
        f = np.zeros(n, dtype=np.uint8)
        f[starts] = 1
        want = oracle.segscan(x, f).astype(np.float32)
        for packed in (True, False):
            z = B.mmv_segscan(xt, flags_dev(f, packed), n=n)
            assert np.array_equal(z.cpu().numpy(), want), (starts, packed)
            out, nseg = B.mmv_segsum(xt, flags_dev(f, packed), n=n)
            assert np.array_equal(out.cpu().numpy()[:int(nseg.item())], oracle.segsum(x, f).astype(np.float32)), (starts, packed)
        if not starts:
            assert np.array_equal(B.mmv_scan(xt, n=n).cpu().numpy(), want)


@pytest.mark.parametrize("n", [300, 60_001, 200_003])
def test_outputs_over_byte_flags(n):
    """Byte flags are packed by a launch of their own before the first result is written, as for long vectors."""
    rng = np.random.default_rng(2390707)
    f = (rng.random(n) < 0.003).astype(np.uint8)
    for dt in ("f32", "i8"):
        x = values(rng, n, dt)
        for shift in (0, 3 * n // 16 * 16):                            # the flags under the first results, under the last ones
            room = torch.zeros(4 * n + 16, dtype=torch.uint8, device="cuda")
            room[shift:shift + n] = dev(f)
            z = room[:4 * n].view(torch.float32 if dt == "f32" else torch.int32)
            B.mmv_segscan(dev(x), room[shift:shift + n], n=n, z=z)
            assert np.array_equal(z.cpu().numpy().astype(np.float64), oracle.segscan(x, f).astype(np.float64))
            room[shift:shift + n] = dev(f)
            _, nseg = B.mmv_segsum(dev(x), room[shift:shift + n], n=n, out=z)
            ref = oracle.segsum(x, f)
            assert int(nseg.item()) == len(ref) and np.array_equal(z.cpu().numpy()[:len(ref)].astype(np.float64), ref.astype(np.float64))


@pytest.mark.parametrize("packed", [True, False])
@pytest.mark.parametrize("dt", list(TYPES))
def test_single_flags_where_more_waves_help(dt, packed):
    """One launch with 1024 threads from so many bytes of values and flags on (MANY_BITS, MANY_BYTES; 7 or 9 KB without flags): both sides of these lines, and the
    start of the last segment at borders of the 128-bit words, just inside and outside what the threads hold from the
    beginning (one word each before the tile), and far back."""
    rng = np.random.default_rng(2390708)
    size = torch.empty(0, dtype=TYPES[dt][0]).element_size()
    per_elem, epl = size + (1 / 8 if packed else 1), 16 // size
    scan_line = ((7 if size == 1 else 9) << 10) // size
    line = int(((MANY_BITS if packed else MANY_BYTES)[size] << 10) / per_elem)
    for n in (scan_line - epl, scan_line - 1, scan_line, line - 1, line + 1, one_launch(dt, per_elem - size) - 3):
        last_tile = (n - 1) // TILE * TILE
        near = 1024 * epl                                              # elements that the threads hold
        at = {1, epl - 1, epl, 5 * epl + 1, TILE - 1, TILE, TILE + epl // 2}
        for edge in (last_tile, last_tile - near, last_tile - 256 * epl, last_tile - near - 128):
            at |= {edge - 1, edge, edge + 1, edge - epl, edge + epl - 1}
        for p in sorted(q for q in at if 0 < q < n):
            f = np.zeros(n, dtype=np.uint8)
            f[p] = 1
            print(dt, packed, n, p, flush=True)
            check(dt, n, packed, f, rng, scan_too=p == 1)


@pytest.mark.parametrize("packed", [True, False])
def test_compress_counts_what_lies_before_every_tile(packed):
    """One selected position at a time, in the words that the threads of a later tile count in their first, second and last round."""
    n = 1 << (20 if packed else 17)
    word = 128 if packed else 16
    for p in (0, word - 1, word, 511 * word, 512 * word - 1, 512 * word, 4 * 512 * word - 1, 4 * 512 * word, 5 * 512 * word + 3, n - 8193, n - 8192, n - 1):
        if p >= n:
            continue
        m = np.zeros(n, dtype=np.uint8)
        m[[p, n - 1]] = 1
        want = np.flatnonzero(m)
        print(packed, p, flush=True)
        out, count = B.mmv_compress(None, flags_dev(m, packed), n)
        assert int(count.item()) == len(want) and np.array_equal(out.cpu().numpy()[:len(want)], want)
