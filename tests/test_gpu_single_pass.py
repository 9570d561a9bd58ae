"""The single-pass kernels of scans and sums, which vectors beyond 2^21 elements or so take, and calls whose output lies over their
flags at any length: where tiles, chunks and rows begin and end, in place, next to values that are not finite."""
import itertools

import numpy as np
import pytest
import torch

import oracle
from paper_2506_23906_amd import binding as B
from paper_2506_23906_amd import workloads as W
from parity_util import check_scan, check_sum, dev, flags_dev, packed_dev, random_values, run_segscan, run_segsum

pytestmark = pytest.mark.gpu
VARIANTS = ["mfma", "shuffle"]
TYPES = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16, "i8": torch.int8, "u8": torch.uint8}
SHORT_TILE = 2048
TILE = 65536          # largest workgroup tile (bytes)


def first_beyond(op, dt):
    """The shortest length that takes the single-pass kernels."""
    code = B._DTYPES[TYPES[dt]]
    for n in (1 << 21, 3 << 20, 1 << 22):
        if B.mmv_tile_elems(op, code, n) == SHORT_TILE and B.mmv_tile_elems(op, code, n + 1) != SHORT_TILE:
            return n + 1
    raise AssertionError("no line found")


def whole_numbers(rng, n, dt):
    x = rng.integers(0, 256, size=n) if dt == "u8" else rng.integers(-3, 4, size=n)
    return x.astype({"f16": np.float16, "i8": np.int8, "u8": np.uint8}.get(dt, np.float32))


def same(got, want):
    assert np.array_equal(got.cpu().numpy().astype(np.float64), want.astype(np.float64))


@pytest.mark.parametrize("variant", VARIANTS)
@pytest.mark.parametrize("dt", list(TYPES))
def test_just_beyond_the_short_vectors(dt, variant):
    """Ragged lengths, both flag formats, workspaces full of garbage, an output array that is too short."""
    rng = np.random.default_rng(2390720)
    code = B._DTYPES[TYPES[dt]]
    for ragged in (0, 1, 31, 33, 2047, 2049, 16383, 16385, 3 * TILE + 77):
        for op in (B.MMV_OP_SEGSCAN, B.MMV_OP_SEGSUM, B.MMV_OP_SCAN):
            n = first_beyond(op, dt) + ragged
            x = whole_numbers(rng, n, dt)
            xt = dev(x).to(TYPES[dt])
            for density in (0.0, 0.05, 1.0)[:1 if op == B.MMV_OP_SCAN else 3]:
                packed = bool((ragged + int(20 * density)) % 2)
                f = ((rng.random(n, dtype=np.float32) < density) * rng.integers(1, 256, size=n)).astype(np.uint8)
                f = (f != 0).astype(np.uint8) if packed else f
                ff = B.MMV_FLAGS_PACKED32 if packed else B.MMV_FLAGS_U8
                print(dt, variant, op, n, density, flush=True)
                ws = torch.full((B.mmv_workspace_bytes(op, code, ff, n),), 0xFF, dtype=torch.uint8, device="cuda")
                if op == B.MMV_OP_SCAN:
                    same(B.mmv_scan(xt, n=n, variant=variant, ws=ws), oracle.scan(x))
                elif op == B.MMV_OP_SEGSCAN:
                    same(B.mmv_segscan(xt, flags_dev(f, packed), n=n, variant=variant, ws=ws), oracle.segscan(x, f))
                else:
                    ref = oracle.segsum(x, f)
                    cap = len(ref) - len(ref) // 3
                    out = torch.full((cap + 64,), -77, dtype=B._OUT_DTYPE[code], device="cuda")
                    _, nseg = B.mmv_segsum(xt, flags_dev(f, packed), n=n, out=out[:cap], variant=variant, ws=ws)
                    assert int(nseg.item()) == len(ref) and bool((out[cap:] == -77).all())
                    same(out[:cap], ref[:cap])
                assert B.mmv_workspace_status(ws) == 0


@pytest.mark.parametrize("variant", VARIANTS)
@pytest.mark.parametrize("dt", list(TYPES))
def test_short_lengths_with_the_flags_under_the_output(dt, variant):
    """Byte flags are packed before the first result is written, and no other kernel than the single-pass ones may take such a
    call: one tile, a few, ragged ones, real values (whole ones in bf16, which the oracle does not know)."""
    rng = np.random.default_rng(2390721)
    code = B._DTYPES[TYPES[dt]]
    for n in (1, 2, 31, 32, 33, 63, 64, 65, 1023, 1024, 1025, 2047, 2048, 2049, 16383, 16384, 16385, TILE - 1, TILE, TILE + 1, 3 * TILE + 77, 16 * TILE + 5):
        for density in (0.0, 0.002, 0.05, 0.5, 1.0):
            x = whole_numbers(rng, n, dt) if dt == "bf16" else random_values(rng, n, {"f16": np.float16, "i8": np.int8, "u8": np.uint8}.get(dt, np.float32))
            f = ((rng.random(n) < density) * rng.integers(1, 256, size=n)).astype(np.uint8)
            print(dt, variant, n, density, flush=True)
            xt = dev(x).to(TYPES[dt])
            room = torch.zeros(4 * n + 16, dtype=torch.uint8, device="cuda")
            z = room[:4 * n].view(B._OUT_DTYPE[code])
            at = 0 if n % 2 else 3 * n // 16 * 16                          # under the first results, under the last ones
            room[at:at + n] = dev(f)
            B.mmv_segscan(xt, room[at:at + n], n=n, z=z, variant=variant)
            check_scan(z.cpu().numpy(), x, f)
            room[at:at + n] = dev(f)
            _, nseg = B.mmv_segsum(xt, room[at:at + n], n=n, out=z, variant=variant)
            check_sum(z.cpu().numpy(), int(nseg.item()), x, f)


@pytest.mark.parametrize("variant", VARIANTS)
def test_every_flag_pattern_n10(variant):
    """All 2^n flag patterns, n <= 10, laid end to end over and over: at every place in a row, a chunk and a tile."""
    for n in (3, 7, 10):
        pats = np.array(list(itertools.product((0, 1), repeat=n)), dtype=np.uint8)
        pats[:, 0] = 1
        reps = (1 << 21) // pats.size + 2
        f = np.tile(pats.reshape(-1), reps)
        x = np.tile(np.arange(1, n + 1, dtype=np.int8) * 5 - 17, len(pats) * reps)
        print(variant, n, flush=True)
        check_scan(run_segscan(x, f, variant), x, f)
        out, nseg = run_segsum(x, f, variant)
        check_sum(out, nseg, x, f)
        xf = x.astype(np.float32)
        assert np.array_equal(run_segscan(xf, f, variant), oracle.segscan(xf, f).astype(np.float32))


@pytest.mark.parametrize("variant", VARIANTS)
@pytest.mark.parametrize("dt", list(TYPES))
def test_single_flags_at_borders(dt, variant):
    rng = np.random.default_rng(2390722)
    n = first_beyond(B.MMV_OP_SEGSCAN, dt) + 2 * TILE + 100
    n_sum = first_beyond(B.MMV_OP_SEGSUM, dt) + 2 * TILE + 100
    x = whole_numbers(rng, n_sum, dt)
    xt = dev(x).to(TYPES[dt])
    for p in (0, 1, 31, 32, 63, 64, 1023, 1024, 2047, 2048, 2049, 16383, 16384, 32768, 32769, TILE - 1, TILE, 20 * TILE + 7, n - 2049, n - 33, n - 2, n - 1):
        f = np.zeros(n_sum, dtype=np.uint8)
        f[p] = 1
        print(dt, variant, p, flush=True)
        same(B.mmv_segscan(xt, packed_dev(f[:n]), n=n, variant=variant), oracle.segscan(x[:n], f[:n]))
        out, nseg = B.mmv_segsum(xt, packed_dev(f), n=n_sum, variant=variant)
        ref = oracle.segsum(x, f)
        assert int(nseg.item()) == len(ref)
        same(out[:len(ref)], ref)


@pytest.mark.parametrize("dtype", [np.int8, np.float16, np.float32])
def test_shift_invariance(dtype):
    """Prepending k single-element segments moves every row and tile border."""
    rng = np.random.default_rng(2390723)
    n = (1 << 21) + TILE + 100
    x = random_values(rng, n, dtype)
    f = W.uniform_density_flags(n, 0.01, seed=5)
    for k in (1, 3, 31, 32, 33, 64, 2047, 2049):
        xs = np.concatenate([random_values(rng, k, dtype), x])
        fs = np.concatenate([np.ones(k, dtype=np.uint8), f])
        print("shift", dtype.__name__, k, flush=True)
        check_scan(run_segscan(xs, fs), xs, fs)


@pytest.mark.parametrize("variant", VARIANTS)
def test_in_place_fp32(variant):
    x, f = W.scan_sum_f32_bernoulli((1 << 22) + 3 * TILE + 5, seed=8)
    for packed in (True, False):
        xt = dev(x)
        B.mmv_segscan(xt, flags_dev(f, packed), z=xt, variant=variant)
        check_scan(xt.cpu().numpy(), x, f)
    whole = np.random.default_rng(2390724).integers(-3, 4, size=len(x)).astype(np.float32)
    xt = dev(whole)
    B.mmv_scan(xt, z=xt, variant=variant)
    same(xt, oracle.scan(whole))


@pytest.mark.parametrize("variant", VARIANTS)
def test_fp32_chunks_with_every_flag_set(variant):
    """Blocks of 2048 positions that all start segments (stored straight from the loaded registers by the matrix-core variant) between
    ordinary ones, at aligned and unaligned places, with a ragged end, and in place: in a whole chunk of set flags the result is
    the input bit for bit."""
    rng = np.random.default_rng(2390725)
    n = (130 + 37) * 16384 + 2048 * 3 + 777
    x = rng.standard_normal(n, dtype=np.float32)
    f = (rng.random(n) < 0.02).astype(np.uint8)
    for a, b in [(0, 2048), (4096, 4096 + 3 * 2048), (16384 * 5 - 2048, 16384 * 5 + 2048), (100_000, 109_999), (16384 * 20, 16384 * 23),
                 (16384 * 140 + 100, 16384 * 142), (n - 2048 - 777, n - 777), (n - 700, n)]:
        f[a:b] = 1
    whole = np.flatnonzero(f[:n - n % 2048].reshape(-1, 2048).all(axis=1))
    assert len(whole) >= 24

    def check(z):
        check_scan(z, x, f)
        if variant == "mfma":
            for c in whole:
                assert np.array_equal(z[2048 * c:2048 * c + 2048].view(np.uint32), x[2048 * c:2048 * c + 2048].view(np.uint32)), c

    check(run_segscan(x, f, variant))
    xt = dev(x)
    B.mmv_segscan(xt, packed_dev(f), n=n, z=xt, variant=variant)
    check(xt.cpu().numpy())


@pytest.mark.parametrize("variant", VARIANTS)
def test_fp32_segment_starts_hold_their_input_and_non_finite_values_stay_in_their_row(variant):
    """The method subtracts two speculative prefixes of a row of 32.  (1) Every position that starts a segment holds its input bit
    for bit, also right behind a huge value or an infinity; (2) what is not finite stays in the row of the infinity, whose segment
    it ends in; (3) the error behind a huge value is within the rounding of that row's prefix, everything else as accurate as ever."""
    rng = np.random.default_rng(2390726)
    n = (1 << 21) + 3 * 16384 + 1000
    x = (rng.random(n, dtype=np.float32) * 2 - 1).astype(np.float32)
    f = (rng.random(n) < 0.1).astype(np.uint8)
    f[0] = 1
    rows_inf, rows_huge = [700, 64 * 33 + 63, n // 32 - 5], [5, 512 * 40]           # (in a chunk, its last row, the last tile)
    ok = np.ones(n, dtype=bool)
    for r in rows_inf + rows_huge:
        p = 32 * r + 11
        f[p - 3:p + 12] = 0
        f[[p - 3, p + 1, p + 6, 32 * r + 32]] = 1        # a segment of four with it, two right behind it, one in the next row
        x[p] = np.inf if r in rows_inf else 3.0e30
        ok[32 * r:32 * r + 32] = False
    z = run_segscan(x, f, variant)
    with np.errstate(invalid="ignore", over="ignore"):
        ref = oracle.segscan(x, f)
    starts = np.flatnonzero(f)
    assert np.array_equal(z[starts].view(np.uint32), x[starts].view(np.uint32))
    assert np.isinf(z[[32 * r + 11 for r in rows_inf]]).all()
    assert set((np.flatnonzero(~np.isfinite(z)) // 32).tolist()) == set(rows_inf)
    A = oracle.segscan(np.abs(np.where(np.isfinite(x), x, 0).astype(np.float64)), f)
    assert (np.abs(z[ok].astype(np.float64) - ref[ok]) <= 2e-5 * np.maximum(A[ok], 1.0)).all()
    for r in rows_huge:
        row = slice(32 * r, 32 * r + 32)
        assert (np.abs(z[row].astype(np.float64) - ref[row]) <= 2.0 ** -22 * 3.0e30).all()


def test_fp16_subnormal_single_element_segments():
    n = (1 << 21) + 4096
    x = (np.arange(n) % 1023 + 1).astype(np.uint16).view(np.float16)     # every positive subnormal
    f = np.ones(n, dtype=np.uint8)
    for variant in VARIANTS:
        check_scan(run_segscan(x, f, variant), x, f)


def test_random_cases_against_the_oracle():
    rng = np.random.default_rng(2390727)
    for case in range(60):
        dtype = [np.int8, np.float16, np.float32][case % 3]
        n = (1 << 21) + int(2 ** rng.uniform(0, 22.5))
        variant, packed = VARIANTS[rng.integers(0, 2)], bool(rng.integers(0, 2))
        x = random_values(rng, n, dtype)
        kind = rng.integers(0, 3)
        if kind == 0:
            f = (rng.random(n, dtype=np.float32) < 10.0 ** rng.uniform(-6, 0)).astype(np.uint8)
        elif kind == 1:
            f = W.flags_from_lengths(W.draw_lengths_until(rng, n, lambda r, k: r.geometric(1.0 / r.integers(2, 50_000), size=k)), n)
        else:                                                            # dense start, one long run, dense end
            f = np.zeros(n, dtype=np.uint8)
            a, b = sorted(rng.integers(0, n + 1, size=2))
            f[:a], f[b:] = rng.random(a) < 0.5, rng.random(n - b) < 0.5
        print(case, n, np.dtype(dtype).name, variant, packed, kind, flush=True)
        if rng.random() < 0.5:
            check_scan(run_segscan(x, f, variant, packed), x, f)
        else:
            out, nseg = run_segsum(x, f, variant, packed)
            check_sum(out, nseg, x, f)
