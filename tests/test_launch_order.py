"""Which kernels a call launches, in which order, with the HIP run-time replaced by one that only writes them down
(hip_recorder.c): no GPU, no memory behind the addresses."""
import ctypes
import re
import subprocess
import sys
import textwrap

import pytest

from conftest import ROOT

X, F, OUT, WS = 0x10_0000_0000, 0x20_0000_0000, 0x30_0000_0000, 0x40_0000_0000     # far apart: nothing overlaps
BYTES, BITS = 0, 1


@pytest.fixture(scope="module")
def record(tmp_path_factory, libmmvseg_path):
    """record(calls): what each of the calls (statements on `lib`, the loaded library) would have the device do;
    record(calls, grids=True): the launches with their workgroups and the threads of each."""
    so = str(tmp_path_factory.mktemp("hip") / "libhip_recorder.so")
    subprocess.run(["gcc", "-shared", "-fPIC", "-O1", "-Wall", "-o", so, "tests/hip_recorder.c"], cwd=ROOT, check=True, timeout=120)
    child = textwrap.dedent("""
        import ctypes, sys
        rec = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
        rec.recorder_log.restype = ctypes.c_char_p
        lib = ctypes.CDLL(sys.argv[2])
        lib.mmv_workspace_bytes.restype = lib.mmv_spmv_csr_workspace_bytes.restype = ctypes.c_size_t
        u64, vp, size = ctypes.c_uint64, ctypes.c_void_p, ctypes.c_size_t
        for call in sys.stdin.read().split(";"):
            rec.recorder_clear()
            print("status", eval(call))
            print(rec.recorder_log().decode(), end="")
            print("--", flush=True)
        """)

    def run(calls, grids=False):
        res = subprocess.run([sys.executable, "-c", child, so, libmmvseg_path], input=";".join(calls), capture_output=True, text=True, timeout=120)
        assert res.returncode == 0, res.stderr[-2000:]
        out = []
        for block in res.stdout.split("--\n")[:-1]:
            lines = block.strip().split("\n")
            assert lines[0] == "status 0", block
            # "launch _ZN..12short_kernelI..E.. grid block" -> "short_kernel" (events stay as they are)
            names = [re.search(r"\d+([a-z_]+_kernel)", line).group(1) if line.startswith("launch") else line for line in lines[1:]]
            out.append([(name, *map(int, line.split()[2:])) for name, line in zip(names, lines[1:])] if grids else names)
        return out
    return run


def segscan(n, dt, ff, z, x=X, f=F):
    return "lib.mmv_segscan(vp(%d), vp(%d), u64(%d), vp(%d), %d, %d, 0, vp(%d), size(1 << 40), None)" % (x, f, n, z, dt, ff, WS)


def segsum(n, dt, ff, out, cap=None, x=X, f=F):
    return ("lib.mmv_segsum(vp(%d), vp(%d), u64(%d), vp(%d), u64(%d), vp(%d), %d, %d, 0, vp(%d), size(1 << 40), None)" %
            (x, f, n, out, n if cap is None else cap, OUT - 64, dt, ff, WS))


def scan(n, dt, z, x=X):
    return "lib.mmv_scan(vp(%d), u64(%d), vp(%d), %d, 0, vp(%d), size(1 << 40), None)" % (x, n, z, dt, WS)


def compress(n, ff, out, cap=None, x=X, f=F):
    return ("lib.mmv_compress(vp(%d), vp(%d), u64(%d), vp(%d), u64(%d), vp(%d), %d, vp(%d), size(1 << 40), None)" %
            (x, f, n, out, n if cap is None else cap, OUT - 64, ff, WS))


F32, F16, I8 = 0, 1, 3
ONE, TWO = ["short_kernel"], ["short_reduce_kernel", "short_kernel"]
PACK, FILL, COUNT = ["pack_flags_kernel", "seg_kernel"], ["fill_zero_kernel", "seg_kernel"], "count_spans_kernel"


@pytest.mark.parametrize("call,want", [
    # an output of its own: one launch, two, the single-pass kernel
    (segscan(30_000, F32, BYTES, OUT), ONE), (segscan(300_000, F32, BYTES, OUT), TWO), (segscan(3_000_000, F32, BYTES, OUT), PACK),
    (segsum(30_000, F32, BITS, OUT), ONE), (segsum(300_000, I8, BITS, OUT), TWO), (segsum(3_000_000, I8, BITS, OUT), [COUNT, "seg_kernel"]),
    (scan(30_000, I8, OUT), ONE), (scan(3_000_000, I8, OUT), TWO), (scan(30_000_000, I8, OUT), FILL),
    # outputs that end where an input begins, and begin where one ends
    (segscan(4096, F32, BYTES, X - 4 * 4096), ONE), (segscan(4096, F32, BYTES, F + 4096), ONE), (segscan(4096, F32, BITS, F + 512), ONE),
    (segsum(4096, F32, BYTES, F - 400, cap=100), ONE),
    # a scan over its own values: every thread's results over what it has loaded, not in one launch
    (segscan(30_000, F32, BYTES, X), TWO), (segscan(300_000, F32, BITS, X), TWO), (scan(30_000, F32, X), TWO),
    # over other values, over flags; sums over either: byte flags are packed before anything is written, as for long vectors
    (segscan(30_000, F32, BYTES, X + 16), PACK), (segscan(300_000, I8, BYTES, F), PACK), (segscan(30_000, I8, BYTES, F + 29_984), PACK),
    (segscan(30_000, I8, BITS, F), FILL), (segscan(30_000, F16, BYTES, F - 4 * 30_000 + 16), PACK), (scan(30_000, F32, X + 16), FILL),
    (segsum(30_000, F32, BYTES, X), [COUNT, "stream_kernel"]), (segsum(30_000, I8, BYTES, X), [COUNT, "seg_kernel"]),
    (segsum(300_000, F32, BYTES, F, cap=1), [COUNT, "stream_kernel"]), (segsum(30_000, I8, BITS, F + 3744, cap=5), [COUNT, "seg_kernel"]),
    (segsum(30_000, F16, BYTES, F - 416, cap=105), [COUNT, "seg_kernel"]),
    # COMPRESS: one launch only with an output apart from the mask and from x
    (compress(30_000, BYTES, OUT), ["compress_kernel"]), (compress(30_000, BITS, OUT), ["compress_kernel"]),
    (compress(30_000, BYTES, F), ["fill_zero_kernel", "compress_kernel"]), (compress(30_000, BITS, X), ["fill_zero_kernel", "compress_kernel"]),
    (compress(30_000, BITS, X + 119_984, cap=7), ["fill_zero_kernel", "compress_kernel"]),
    (compress(30_000, BYTES, F - 16, cap=4), ["compress_kernel"]), (compress(30_000, BITS, OUT, x=0), ["compress_kernel"]),
])
def test_overlapping_outputs_take_the_launches_they_are_safe_in(record, call, want):
    assert record([call]) == [want]


@pytest.mark.parametrize("call,want", [
    (segscan(65_536, F32, BYTES, OUT), ONE), (segscan(65_537, F32, BYTES, OUT), TWO), (segsum(163_840, I8, BYTES, OUT), ONE), (segsum(163_841, I8, BYTES, OUT), TWO),
    (segsum(109_226, F16, BYTES, OUT), ONE), (segsum(109_227, F16, BYTES, OUT), TWO), (segscan(154_176, F16, BITS, OUT), ONE), (segscan(154_240, F16, BITS, OUT), TWO),
    (scan(163_840, F16, OUT), ONE), (scan(163_841, F16, OUT), TWO), (scan(3 << 20, F16, OUT), TWO), (scan((3 << 20) + 1, F16, OUT), FILL),
    (segscan(1 << 21, F16, BYTES, OUT), TWO), (segscan((1 << 21) + 1, F16, BYTES, OUT), PACK), (segscan((1 << 21) + 1, F32, BITS, OUT), FILL),
    (segsum(1 << 21, F16, BITS, OUT), TWO), (segsum(3 << 20, F32, BITS, OUT), TWO), (segsum((3 << 20) + 1, F32, BITS, OUT), [COUNT, "stream_kernel"]),
])
def test_lines_between_the_forms(record, call, want):
    assert record([call]) == [want]


@pytest.mark.parametrize("call,threads", [
    (segscan(20_000, F32, BITS, OUT), 256), (segscan(65_536, F32, BITS, OUT), 256), (segscan(71_500, F32, BITS, OUT), 1024),
    (segsum(32_767, F32, BYTES, OUT), 256), (segsum(32_768, F32, BYTES, OUT), 1024), (segsum(40_966, F16, BITS, OUT), 256),
    (segsum(115_600, F16, BITS, OUT), 256), (segsum(115_700, F16, BITS, OUT), 1024), (segscan(43_690, F16, BYTES, OUT), 256), (segscan(43_691, F16, BYTES, OUT), 1024),
    (segscan(87_300, I8, BITS, OUT), 256), (segscan(87_400, I8, BITS, OUT), 1024), (segsum(40_959, I8, BYTES, OUT), 256),
    (segsum(40_960, I8, BYTES, OUT), 1024), (scan(2_303, F32, OUT), 256), (scan(2_304, F32, OUT), 1024),
    (scan(7_167, I8, OUT), 256), (scan(7_168, I8, OUT), 1024),
])
def test_threads_of_the_one_launch(record, call, threads):
    """The twelve waves more that read what lies before a tile pay only where a workgroup may have much to read."""
    assert record([call], grids=True)[0][0][::2] == ("short_kernel", threads)


@pytest.mark.parametrize("call,want", [
    (segscan(30_000, F32, BYTES, OUT), ["event 5", *ONE, "event 7"]), (segscan(300_000, F32, BITS, OUT), ["event 5", *TWO, "event 7"]),
    (segsum(300_000, I8, BYTES, OUT), ["event 5", *TWO, "event 7"]), (scan(300_000, F16, OUT), ["event 5", *TWO, "event 7"]),
    (segscan(3_000_000, F32, BYTES, OUT), [PACK[0], "event 5", PACK[1], "event 7"]),
    (segsum(3_000_000, I8, BITS, OUT), [COUNT, "event 5", "seg_kernel", "event 7"]),
    (compress(30_000, BITS, OUT), ["event 5", "compress_kernel", "event 7"]),
])
def test_kernel_events_stand_around_all_that_reads_the_inputs(record, call, want):
    """... and behind what only resets the workspace, packs or counts flags."""
    assert record(["lib.mmv_set_kernel_events(vp(5), vp(7))", call])[1] == want


@pytest.mark.parametrize("n_rows,nnz,tiles,helpers", [
    (65_536, 1 << 20, 128, 8), (16_384, 1 << 20, 128, 0), (16_385, 1 << 20, 128, 3), (1 << 20, 1 << 25, 763, 128), (44_032, 1 << 25, 763, 0),
    (44_033, 1 << 25, 763, 6), (1 << 20, (1 << 20) // 3, 43, 128), (49_152, 16_384, 2, 0), (49_152, 16_385, 3, 6),
])
def test_rows_of_a_csr_tile_are_shared(record, n_rows, nnz, tiles, helpers):
    """One workgroup per tile is not enough where nearly all rows may start in one: a workgroup for every 8192 rows besides, from where a
    tile can hold more than 16384 rows, more rows than entries and twice its part."""
    prepare = "lib.mmv_spmv_csr_prepare(u64(%d), u64(100), u64(%d), vp(%d), vp(%d), vp(%d), size(1 << 40), None)" % (n_rows, nnz, X, F, WS)
    assert record([prepare], grids=True)[0][0] == ("csr_plan_kernel", tiles + helpers, 256)
