"""Scans of fp32 values of any length that the single-pass kernel takes (lane_tile): blocks of 256 elements carried from lane to lane."""
import numpy as np
import pytest
import torch

import oracle
from paper_2506_23906_amd import binding as B
from parity_util import abs_scan, dev, flags_dev

pytestmark = pytest.mark.gpu
BLOCK, WAVE, TILE = 256, 2048, 16384
BORDERS = [1, 3, 4, 255, 256, 257, 511, 2047, 2048, 2049, 16383, 16384, 16385, 32768, 49153]   # lanes, blocks, waves, tiles


def flags_at(n, places):
    f = np.zeros(n, dtype=np.uint8)
    f[[p for p in places if p < n]] = 1
    return f


@pytest.mark.parametrize("packed", [True, False])
@pytest.mark.parametrize("ragged", [1, 3, 255, 258, 2049, 16387])
def test_flags_at_borders_and_the_bound_of_the_error(ragged, packed):
    """A result is rounded where a lane's four values are added up (three times at most, each at most 2^-24 of A, the sum of |x| of its
    segment so far), where the carry into the lane is, and when the two are added: 5 * 2^-24 * A.  What is carried in 64 bits adds
    nothing that shows, and a start receives its input bit for bit."""
    n = (1 << 21) + ragged
    rng = np.random.default_rng(ragged)
    x = rng.uniform(-1, 1, size=n).astype(np.float32)
    patterns = {"none": [], "borders": BORDERS + [n - b for b in BORDERS], "one late": [n - 1], "one in a block": [40 * TILE + 777],
                "a dense block": list(range(5 * TILE + 3 * BLOCK, 5 * TILE + 4 * BLOCK)), "all": range(n), "sparse": np.flatnonzero(rng.random(n) < 1e-3),
                "lanes": np.flatnonzero(rng.random(n) < 0.2)}
    for name, places in patterns.items():
        f = flags_at(n, places)
        print(n, packed, name, flush=True)
        z = B.mmv_segscan(dev(x), flags_dev(f, packed), n=n).cpu().numpy()
        err = np.abs(z.astype(np.float64) - oracle.segscan(x, f))
        assert (err <= 5 * 2.0 ** -24 * abs_scan(x, f)).all(), name
        assert np.array_equal(z[f == 1].view(np.uint32), x[f == 1].view(np.uint32)), name


def test_values_that_are_not_finite_stay_in_their_segment():
    n = (1 << 21) + 77
    rng = np.random.default_rng(5)
    x = rng.integers(-3, 4, size=n).astype(np.float32)
    f = (rng.random(n) < 0.01).astype(np.uint8)
    bad = np.concatenate([[b + d for b in (BLOCK, WAVE, TILE, 2 * TILE) for d in (-1, 0, 1)], rng.integers(0, n, size=200)])
    x[bad] = rng.choice([np.inf, -np.inf, np.nan, 3e38], size=len(bad))
    z = B.mmv_segscan(dev(x), flags_dev(f, True), n=n).cpu().numpy()
    f[0] = 1
    seg = np.cumsum(f)
    touched = np.isin(seg, seg[bad])
    assert np.array_equal(z[~touched], oracle.segscan(np.where(touched, 0, x).astype(np.float32), f)[~touched].astype(np.float32))
    with np.errstate(invalid="ignore", over="ignore"):
        for s in np.unique(seg[bad])[:100]:                    # (in 64 bits, rounded: what overflows 32 bits is infinite)
            i = np.flatnonzero(seg == s)
            want = np.cumsum(x[i].astype(np.float64))
            assert np.array_equal(np.isnan(z[i]), np.isnan(want)), s
            gone = np.flatnonzero(~np.isfinite(want.astype(np.float32)))[:1]     # up to there the segment is finite
            upto = gone[0] if len(gone) else len(i)
            assert (np.abs(z[i][:upto] - want[:upto]) <= 5 * 2.0 ** -24 * np.cumsum(np.abs(x[i][:upto].astype(np.float64)))).all(), s


@pytest.mark.parametrize("op,n,tt", [("segscan", (1 << 21) + 5, torch.float32), ("scan", (1 << 22) + 5, torch.float32), ("segscan", (1 << 24) + 5, torch.bfloat16)])
def test_sums_that_overflow_inside_a_lane_only(op, n, tt):
    """Prefixes are whole multiples of 2^125, at most seven in magnitude: finite, and every sum in 64 bits is exact, while two neighbours
    may add up to fourteen, beyond 32 bits."""
    rng = np.random.default_rng(n)
    for density in (0.0, 1e-5, 1e-3, 0.2) if op == "segscan" else (0.0,):
        f = (rng.random(n, dtype=np.float32) < density).astype(np.uint8)
        for places in (1.0, 1e-4):                             # everywhere; a few, most waves without
            want, start = np.full(n, -7, dtype=np.int64), f.copy()
            start[0] = 1
            even = want[::2]
            new = rng.random(len(even), dtype=np.float32) < places
            even[new] = rng.integers(-7, 8, size=int(new.sum()))
            want[1:-1:2] = (want[:-2:2] + want[2::2]) // 2     # (so that no step is longer than seven)
            x = np.diff(want, prepend=0)
            assert np.abs(x).max() == 7
            x[start == 1] = want[start == 1]
            x = np.ldexp(x.astype(np.float32), 125)
            want = np.ldexp(want.astype(np.float32), 125)
            print(op, n, tt, density, places, flush=True)
            xt = dev(x).to(tt)
            z = B.mmv_scan(xt, n=n) if op == "scan" else B.mmv_segscan(xt, flags_dev(f, True), n=n)
            assert np.array_equal(z.cpu().numpy(), want), (density, places)
            if op == "segscan":                                # the lane's four values from a start inside it on
                lone = np.zeros(n, dtype=np.float32)
                at = np.arange(1, n - 8, 4096 + 5)
                lone[at - 1], lone[at], lone[at + 1], lone[at + 2] = 3e38, -3e38, 2e38, 2e38
                g = f.copy()
                g[at - 1] = g[at] = 1
                g[at + 1] = g[at + 2] = 0                      # (2e38 and 2e38 alone are infinite)
                lt = dev(lone).to(tt)
                z = B.mmv_segscan(lt, flags_dev(g, True), n=n).cpu().numpy()
                low = lt.float().cpu().numpy()
                assert (np.abs(z - oracle.segscan(low, g)) <= 5 * 2.0 ** -24 * abs_scan(low, g)).all()


@pytest.mark.parametrize("ragged", [1, 257, 4097, 32771])
def test_without_flags(ragged):
    """Beyond the short vectors; the carry of every tile comes from all those before it."""
    n = (1 << 22) + ragged
    x = np.random.default_rng(ragged).uniform(-1, 1, size=n).astype(np.float32)
    none = np.zeros(n, dtype=np.uint8)
    xt = dev(x)
    want, bound = oracle.scan(x), 5 * 2.0 ** -24 * abs_scan(x, none)
    for rep in range(3):
        for z in (B.mmv_scan(xt, n=n, variant=("mfma", "shuffle")[rep % 2]), B.mmv_segscan(xt, flags_dev(none, True), n=n)):
            assert (np.abs(z.cpu().numpy().astype(np.float64) - want) <= bound).all()
    B.mmv_scan(xt, n=n, z=xt)                                  # over its own values
    assert (np.abs(xt.cpu().numpy().astype(np.float64) - want) <= bound).all()


@pytest.mark.parametrize("ragged", [1, 4, 255, 257, 300, 2050, 4095, 16385])
def test_nothing_is_written_behind_the_result(ragged):
    """The last block, the waves behind it that have no elements, both kernels; and nothing of the words behind the flags counts."""
    rng = np.random.default_rng(ragged)
    for op, base in (("segscan", 1 << 21), ("scan", 1 << 22)):
        n = base + ragged
        x = rng.integers(-3, 4, size=n).astype(np.float32)
        f = (rng.random(n) < 1e-3).astype(np.uint8) if op == "segscan" else np.zeros(n, dtype=np.uint8)
        room = torch.full((n + 40_000,), 7.0, device="cuda")
        xt = torch.full((n + 40_000,), float("nan"), device="cuda")
        xt[:n] = dev(x)
        if op == "scan":
            B.mmv_scan(xt[:n], n=n, z=room[:n])
        else:
            bits = torch.full(((n + 31) // 32 + 2000,), -1, dtype=torch.int32, device="cuda")
            bits[:(n + 31) // 32] = flags_dev(f, True)[:(n + 31) // 32]
            B.mmv_segscan(xt[:n], bits[:(n + 31) // 32], n=n, z=room[:n])
        assert np.array_equal(room[:n].cpu().numpy(), oracle.segscan(x, f).astype(np.float32)), op
        assert bool((room[n:] == 7.0).all()), op


@pytest.mark.parametrize("ragged", [1, 2, 7, 259, 2051, 16386])
@pytest.mark.parametrize("tt", [torch.float16, torch.bfloat16])
def test_16_bit_values(tt, ragged):
    """Segmented scans just above 2^24 elements.  A lane's four values are added up in 32 bits (three roundings at most, each at most
    2^-24 of A), the rest in 64, and the result is rounded once: 4 * 2^-24 * A.  Nothing behind the inputs counts, nothing is written
    behind the result."""
    n = (1 << 24) + ragged
    rng = np.random.default_rng(ragged)
    room, words = torch.full((n + 40_000,), 7.0, device="cuda"), (n + 31) // 32
    xt = torch.full((n + 40_000,), float("nan"), device="cuda", dtype=tt)
    xt[:n] = dev(rng.standard_normal(n, dtype=np.float32)).to(tt)
    x = xt[:n].float().cpu().numpy()
    for places in ([], BORDERS + [n - b for b in BORDERS], np.flatnonzero(rng.random(n, dtype=np.float32) < 0.2), range(n)):
        f = flags_at(n, places)
        print(tt, n, len(places), flush=True)
        bits = torch.full((words + 2000,), -1, dtype=torch.int32, device="cuda")
        bits[:words] = flags_dev(f, True)[:words]
        z = B.mmv_segscan(xt[:n], bits[:words], n=n, z=room[:n]).cpu().numpy()
        assert (np.abs(z.astype(np.float64) - oracle.segscan(x, f)) <= 4 * 2.0 ** -24 * abs_scan(x, f)).all()
        assert np.array_equal(z[f == 1].view(np.uint32), x[f == 1].view(np.uint32))
        assert bool((room[n:] == 7.0).all())
