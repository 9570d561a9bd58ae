"""The work that the performance of this library is measured on.

Every case is one call of a public entry point of paper_2506_23906_amd.binding, as a program calls it that
keeps its workspace and its output arrays: segmented scan and segmented sum, the unsegmented scan, COMPRESS,
and the sparse matrix-vector product (COO, CSR, in one step and on a prepared matrix).

A case is a dict of plain values:
  op       segscan | segsum | scan | compress | spmv_coo | spmv_csr | spmv_csr_run
  dtype    i8 | u8 (bytes under exclusive or) | f16 | bf16 | f32      (compress: i32 | f32; SpMV is fp32)
  n        elements (SpMV: n_rows = n_cols = n)
  flags    bits | bytes: the encoding of the segment starts (compress: of the mask)
  segs     uniform (lengths 1 .. size) | geometric (mean `size`) | density (each position with probability `size`)
           | none (one segment) | regimes (half the vector all starts, a quarter one segment, the rest short ones)
  variant  mfma (the default of every call) | shuffle
  SpMV     kind zipf (nnz entries in rows of Zipf(1.5) lengths up to `cap`, many rows empty, columns uniform) or
           attention (blocks of `block`, `rand` random blocks per block row, 2 global and 3 window blocks)
"""
import math

import torch

from paper_2506_23906_amd import binding as B

_DT = {"i8": torch.int8, "u8": torch.uint8, "f16": torch.float16, "bf16": torch.bfloat16, "f32": torch.float32,
       "i32": torch.int32}
_SIZE = {"i8": 1, "u8": 1, "f16": 2, "bf16": 2, "f32": 4, "i32": 4}
_CODE = {"i8": B.MMV_I8_I32, "u8": B.MMV_U8_XOR, "f16": B.MMV_F16_F32, "bf16": B.MMV_BF16_F32, "f32": B.MMV_F32_F32}


def listed():
    def seg(name, op, dtype, n, flags, segs, size, variant="mfma"):
        return {"name": name, "op": op, "dtype": dtype, "n": n, "flags": flags, "segs": segs, "size": float(size), "variant": variant}

    def spmv(name, op, kind, n, nnz=0, cap=0, block=0, rand=0):
        return {"name": name, "op": op, "kind": kind, "n": n, "nnz": nnz, "cap": cap, "block": block, "rand": rand, "variant": "mfma"}

    return [
        # a small vector inside a larger program, with the flags as a byte mask: launches and latency
        seg("segscan_f32_small", "segscan", "f32", 65536, "bytes", "density", 1 / 64),
        # 16-bit values, one byte per flag, an odd length: the ordinary call of a program that has a mask
        seg("segscan_f16_bytes", "segscan", "f16", 20_000_003, "bytes", "uniform", 512),
        # the benchmark's own workload: bytes to int32, bit-packed flags, 2^28 elements
        seg("segscan_i8_large", "segscan", "i8", 1 << 28, "bits", "uniform", 4096),
        # fp32 over the three extremes of segment lengths at once (all starts, one segment, short segments)
        seg("segscan_f32_regimes", "segscan", "f32", 1 << 27, "bits", "regimes", 64),
        # sums of short segments of 16-bit values, one round of workgroups
        seg("segsum_f16_mid", "segsum", "f16", 1 << 24, "bits", "geometric", 32),
        # sums of fp32 values, ragged length, byte flags
        seg("segsum_f32_bytes", "segsum", "f32", 100_000_001, "bytes", "density", 0.01),
        # sums of bytes over a long vector
        seg("segsum_i8_large", "segsum", "i8", 1 << 28, "bits", "density", 0.001),
        # running sum of an fp32 vector
        seg("scan_f32", "scan", "f32", 50_000_017, "bits", "none", 0),
        # selection of a third of a vector by a byte mask
        seg("compress_f32_bytes", "compress", "f32", 1 << 26, "bytes", "density", 0.3),
        # a matrix multiplied once: scattered columns, rows of very different lengths, most of them empty
        spmv("spmv_coo_zipf", "spmv_coo", "zipf", 1 << 20, nnz=1 << 25, cap=1 << 14),
        # blocked sparse attention, the mask used once
        spmv("spmv_csr_attention", "spmv_csr", "attention", 65536, block=16, rand=4),
        # ... and a larger one multiplied many times
        spmv("spmv_csr_run_attention", "spmv_csr_run", "attention", 65536, block=64, rand=8),
    ]


def draw(rng):
    def log_uniform(a, b):
        return math.exp(rng.uniform(math.log(a), math.log(b)))

    op = rng.choice(["segscan", "segscan", "segscan", "segsum", "segsum", "segsum", "scan", "compress",
                     "spmv_coo", "spmv_csr", "spmv_csr", "spmv_csr_run"])
    variant = "shuffle" if rng.random() < 0.2 else "mfma"
    if op.startswith("spmv"):
        if op != "spmv_coo" and rng.random() < 0.6:
            block = rng.choice([2, 4, 16, 64])
            n = block * int(log_uniform(4096, 65536) / block)
            return {"op": op, "kind": "attention", "n": n, "nnz": 0, "cap": 0, "block": block,
                    "rand": rng.choice([2, 4, 8]), "variant": variant}
        n = int(log_uniform(1000, 1 << 20))
        nnz = int(min(1 << 25, n * log_uniform(1.0, 64.0)))
        return {"op": op, "kind": "zipf", "n": n, "nnz": nnz, "cap": rng.choice([512, 4096, 1 << 14]), "block": 0,
                "rand": 0, "variant": variant}
    n = int(log_uniform(2000, 1 << 28))
    if rng.random() < 0.25:
        n = 1 << max(11, min(28, round(math.log2(n))))
    if op == "compress":
        dtype = rng.choice(["f32", "i32"])
        n = min(n, 1 << 27)
    else:
        dtype = rng.choice(["i8", "f16", "bf16", "f32", "f32"])
        if op == "segscan" and rng.random() < 0.1:
            dtype, variant = "u8", "shuffle"            # the variant that the header names for this type
        n = min(n, int(1.35e9 / (_SIZE[dtype] + 5)))     # no more bytes than the largest listed case
    segs, size = rng.choice([("uniform", log_uniform(8, 8192)), ("geometric", log_uniform(4, 2000)),
                             ("density", log_uniform(1e-4, 0.5)), ("density", log_uniform(1e-4, 0.5)), ("none", 0.0)])
    if op == "segsum":                                   # a good number of sums, so that their relative error means something
        size = max(size, 64 / n) if segs == "density" else min(size, n / 64) if segs != "none" else 0.01
        segs = "density" if segs == "none" else segs
    if op == "compress":
        segs, size = "density", log_uniform(1e-3, 0.9)
    if op == "scan":
        segs, size = "none", 0.0
    return {"op": op, "dtype": dtype, "n": n, "flags": rng.choice(["bits", "bytes"]), "segs": segs, "size": float(size),
            "variant": variant}


# ---- inputs -------------------------------------------------------------------------------------------------------

def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _uniform01(n, g):
    return torch.rand(n, device="cuda", generator=g)


def _lengths_to_flags(f, lengths):
    starts = torch.cumsum(lengths, 0) - lengths
    f[starts[starts < f.numel()]] = 1


def _flags(case, g):
    """One byte per element, 1 at the first element of every segment (compress: at the selected entries)."""
    n, segs, size = case["n"], case["segs"], case["size"]
    f = torch.zeros(n, dtype=torch.uint8, device="cuda")
    if segs == "density":
        for a in range(0, n, 1 << 26):                   # in pieces: keeps the temporaries small
            b = min(n, a + (1 << 26))
            f[a:b] = _uniform01(b - a, g) < size
    elif segs == "uniform":
        m = max(1, int(size))
        k = int(2.0 * n / (m + 1) * 1.1) + 4096
        _lengths_to_flags(f, torch.randint(1, m + 1, (k,), device="cuda", generator=g))
    elif segs == "geometric":
        k = int(n / size * 1.1) + 4096
        u = _uniform01(k, g).double().clamp_(min=1e-12)
        _lengths_to_flags(f, (torch.log(u) / math.log1p(-1.0 / size)).ceil().clamp_(min=1).long())
    elif segs == "regimes":
        half, quarter = n // 2, n // 4
        f[:half + 1] = 1
        tail = f[half + quarter:]
        m = max(1, int(size))
        _lengths_to_flags(tail, torch.randint(1, m + 1, (int(2.0 * tail.numel() / (m + 1) * 1.1) + 4096,), device="cuda", generator=g))
    if case["op"] != "compress":
        f[0] = 1
    return f


def _pack(f):
    """Bit (i mod 32) of 32-bit word floor(i / 32)."""
    n = f.numel()
    words = torch.empty((n + 31) // 32, dtype=torch.int32, device="cuda")
    weights = (2 ** torch.arange(32, device="cuda", dtype=torch.int64))
    step = 1 << 25
    for a in range(0, n, step):
        b = min(n, a + step)
        part = torch.zeros((b - a + 31) // 32 * 32, dtype=torch.int64, device="cuda")
        part[:b - a] = f[a:b]
        w = (part.view(-1, 32) * weights).sum(1)
        words[a // 32:a // 32 + w.numel()] = torch.where(w >= 2 ** 31, w - 2 ** 32, w).int()
    return words


def _values(case, g):
    n, dtype = case["n"], case["dtype"]
    if dtype == "i8":
        return torch.randint(-8, 9, (n,), dtype=torch.int8, device="cuda", generator=g)
    if dtype == "u8":
        return torch.randint(0, 256, (n,), dtype=torch.uint8, device="cuda", generator=g)
    if dtype == "i32":
        return torch.randint(-2 ** 31, 2 ** 31, (n,), dtype=torch.int32, device="cuda", generator=g)
    if dtype == "f32" and case["op"] != "compress":
        return _uniform01(n, g) * 2 - 1
    return torch.randn(n, device="cuda", generator=g).to(_DT[dtype])


def _zipf_lengths(case, g):
    n, cap = case["n"], min(case["cap"], case["n"])
    k = torch.arange(1, cap + 1, device="cuda", dtype=torch.float64)
    p = k ** -1.5
    q = min(1.0, case["nnz"] / (n * float((k * p).sum() / p.sum())))
    cdf = torch.cumsum(p, 0) / p.sum()
    lengths = torch.searchsorted(cdf, _uniform01(n, g).double()).clamp_(max=cap - 1) + 1
    lengths[_uniform01(n, g) >= q] = 0
    if int(lengths.sum()) == 0:
        lengths[0] = 1
    return lengths


def _attention(case, g):
    """Row lengths and columns: per block row 2 global, 3 window (clipped) and `rand` random block columns, each
    once; the first two block rows are full."""
    n, block = case["n"], case["block"]
    nb = n // block
    i = torch.arange(nb, device="cuda").view(-1, 1)
    window = i + torch.arange(-1, 2, device="cuda").view(1, -1)
    cand = torch.cat([torch.arange(2, device="cuda").view(1, -1).expand(nb, 2), window,
                      torch.randint(0, nb, (nb, case["rand"]), device="cuda", generator=g)], 1)
    cand = torch.where((cand < 0) | (cand >= nb), torch.full_like(cand, nb), cand)     # outside the matrix
    cand = torch.sort(cand, 1).values
    keep = cand < nb
    keep[:, 1:] &= cand[:, 1:] != cand[:, :-1]
    per = keep.sum(1)
    per[:2] = nb
    blocks = torch.cat([torch.arange(nb, device="cuda").repeat(2), cand[2:][keep[2:]]])   # block columns, block row by block row
    lengths = (per * block).repeat_interleave(block)
    first = torch.cumsum(per, 0) - per                   # first block column of a block row in `blocks`
    rowptr = torch.cumsum(lengths, 0) - lengths
    nnz = int(lengths.sum())
    col = torch.empty(nnz, dtype=torch.int32, device="cuda")
    step = 1 << 26
    ends = rowptr + lengths
    for a in range(0, nnz, step):
        e = torch.arange(a, min(nnz, a + step), device="cuda")
        r = torch.searchsorted(ends, e, right=True)
        within = e - rowptr[r]
        col[a:a + e.numel()] = (blocks[first[r // block] + within // block] * block + within % block).int()
    return lengths, col


def _spmv_inputs(case, seed):
    g = _generator(seed)
    n = case["n"]
    if case["kind"] == "zipf":
        lengths = _zipf_lengths(case, g)
        col = torch.randint(0, n, (int(lengths.sum()),), dtype=torch.int32, device="cuda", generator=g)
    else:
        lengths, col = _attention(case, g)
    nnz = col.numel()
    val = torch.randn(nnz, device="cuda", generator=g)
    x = torch.randn(n, device="cuda", generator=g)
    rowptr = torch.zeros(n + 1, dtype=torch.int32, device="cuda")
    rowptr[1:] = torch.cumsum(lengths, 0).int()
    row = None
    if case["op"] == "spmv_coo":
        row = torch.arange(n, device="cuda", dtype=torch.int32).repeat_interleave(lengths)
    return rowptr, row, col, val, x


def _seg_inputs(case, seed):
    g = _generator(seed)
    x = _values(case, g)
    return x, (None if case["op"] == "scan" else _flags(case, g))


def prepare(case, seed):
    op = case["op"]
    if op.startswith("spmv"):
        rowptr, row, col, val, x = _spmv_inputs(case, seed)
        n = case["n"]
        s = {"case": case, "rowptr": rowptr, "row": row, "col": col, "val": val, "x": x,
             "y": torch.empty(n, dtype=torch.float32, device="cuda")}
        if op == "spmv_coo":
            s["ws"] = B.new_workspace(B.MMV_OP_SPMV_COO, B.MMV_F32_F32, B.MMV_FLAGS_PACKED32, val.numel())
        elif op == "spmv_csr":
            s["ws"] = B.workspace(B.mmv_spmv_csr_workspace_bytes(n, val.numel()))
        else:
            s["ws"] = B.mmv_spmv_csr_prepare(n, n, rowptr, col)
        return s
    x, f = _seg_inputs(case, seed)
    n = case["n"]
    s = {"case": case, "x": x}
    ff = B.MMV_FLAGS_PACKED32
    if f is not None:
        ff = B.MMV_FLAGS_U8 if case["flags"] == "bytes" else B.MMV_FLAGS_PACKED32
        s["flags"] = f if case["flags"] == "bytes" else _pack(f)
    if op == "segscan":
        s["z"] = torch.empty(n, dtype=torch.float32 if x.dtype.is_floating_point else torch.int32, device="cuda")
        s["ws"] = B.new_workspace(B.MMV_OP_SEGSCAN, _CODE[case["dtype"]], ff, n)
    elif op == "scan":
        s["z"] = torch.empty(n, dtype=torch.float32 if x.dtype.is_floating_point else torch.int32, device="cuda")
        s["ws"] = B.new_workspace(B.MMV_OP_SCAN, _CODE[case["dtype"]], ff, n)
    elif op == "segsum":
        s["out"] = torch.zeros(_capacity(case), dtype=torch.float32 if x.dtype.is_floating_point else torch.int32, device="cuda")
        s["nseg"] = torch.empty(1, dtype=torch.int64, device="cuda")
        s["ws"] = B.new_workspace(B.MMV_OP_SEGSUM, _CODE[case["dtype"]], ff, n)
    else:
        s["out"] = torch.zeros(_capacity(case), dtype=x.dtype, device="cuda")
        s["count"] = torch.empty(1, dtype=torch.int64, device="cuda")
        s["ws"] = B.new_workspace(B.MMV_OP_COMPRESS, B.MMV_I8_I32, ff, n)
    return s


def run(s):
    case = s["case"]
    op, variant = case["op"], case["variant"]
    n = case["n"]
    if op == "segscan":
        return B.mmv_segscan(s["x"], s["flags"], n=n, z=s["z"], variant=variant, ws=s["ws"])
    if op == "segsum":
        return B.mmv_segsum(s["x"], s["flags"], n=n, out=s["out"], nseg=s["nseg"], variant=variant, ws=s["ws"])
    if op == "scan":
        return B.mmv_scan(s["x"], n=n, z=s["z"], variant=variant, ws=s["ws"])
    if op == "compress":
        return B.mmv_compress(s["x"], s["flags"], n, out=s["out"], count=s["count"], ws=s["ws"])
    if op == "spmv_coo":
        return B.mmv_spmv_coo(n, n, s["row"], s["col"], s["val"], s["x"], y=s["y"], variant=variant, ws=s["ws"])
    if op == "spmv_csr":
        return B.mmv_spmv_csr(n, n, s["rowptr"], s["col"], s["val"], s["x"], y=s["y"], variant=variant, ws=s["ws"])
    return B.mmv_spmv_csr_run(n, n, s["rowptr"], s["col"], s["val"], s["x"], s["ws"], y=s["y"], variant=variant)


# ---- what a pass cannot do without ---------------------------------------------------------------------------------

def _expected_segments(case):
    n, segs, size = case["n"], case["segs"], case["size"]
    if segs == "uniform":
        return max(1.0, 2.0 * n / (max(1, int(size)) + 1))
    if segs == "geometric":
        return max(1.0, n / size)
    if segs == "density":
        return max(1.0, n * size)
    if segs == "regimes":
        return n / 2 + n / 4 * 2.0 / (max(1, int(size)) + 1)
    return 1.0


def _capacity(case):
    """Room that a program gives to an output whose length it knows only roughly."""
    k = _expected_segments(case)
    return int(min(case["n"], 1.02 * k + 8.0 * math.sqrt(k) + 64))


def _padded(v, case):
    out = torch.zeros(_capacity(case), dtype=v.dtype, device=v.device)
    out[:v.numel()] = v
    return out


def _expected_nnz(case):
    n = case["n"]
    if case["kind"] == "zipf":
        cap = min(case["cap"], n)
        a = sum(k ** -0.5 for k in range(1, cap + 1))
        b = sum(k ** -1.5 for k in range(1, cap + 1))
        return min(float(case["nnz"]), n * a / b)
    block, nb = case["block"], case["n"] // case["block"]
    return float(block) * block * (2 * nb + (nb - 2) * min(nb, 5 + case["rand"]))


def work(case):
    op, n = case["op"], case["n"]
    if op.startswith("spmv"):
        nnz = _expected_nnz(case)
        # values, columns and rows (COO: an index per entry, CSR: pointers), x once, y once
        return {"bytes": nnz * (12.0 if op == "spmv_coo" else 8.0) + 4.0 * n + 4.0 * n + (0.0 if op == "spmv_coo" else 4.0 * n),
                "flops": 2.0 * nnz}
    flags = 0.0 if op == "scan" else (n if case["flags"] == "bytes" else n / 8.0)
    if op in ("segscan", "scan"):
        return {"bytes": n * (_SIZE[case["dtype"]] + 4.0) + flags, "flops": float(n)}
    k = _expected_segments(case)
    if op == "segsum":
        return {"bytes": n * float(_SIZE[case["dtype"]]) + flags + 4.0 * k, "flops": float(n)}
    return {"bytes": flags + 8.0 * k, "flops": float(n)}


# ---- results in 64 bits ---------------------------------------------------------------------------------------------

def _sums_between(wide, ends):
    """Sums of consecutive pieces of `wide` that end before the positions `ends`, as differences of its running sums
    (in 64 bits their rounding is nine digits below that of a sum in 32 bits)."""
    c = torch.zeros(wide.numel() + 1, dtype=wide.dtype, device=wide.device)
    torch.cumsum(wide, 0, out=c[1:])
    return torch.diff(c[ends], prepend=c[:1])


def exact(case, seed):
    op = case["op"]
    if op.startswith("spmv"):
        rowptr, _, col, val, x = _spmv_inputs(case, seed)
        return _sums_between(val.double() * x[col.long()].double(), rowptr[1:].long())
    x, f = _seg_inputs(case, seed)
    if op == "compress":
        sel = _padded(x[f.bool()], case)
        return (sel.double() if x.dtype.is_floating_point else sel.long()), f.sum().view(1).long()
    if case["dtype"] == "u8":                            # exclusive or: parities of the eight bit planes
        n = case["n"]
        z = torch.zeros(n, dtype=torch.int32, device="cuda")
        f = f.clone()
        f[0] = 1
        starts = torch.nonzero(f).view(-1)
        lengths = torch.diff(starts, append=torch.tensor([n], device="cuda"))
        for bit in range(8):
            c = torch.cumsum(((x >> bit) & 1).int(), 0, dtype=torch.int32)
            before = torch.where(starts > 0, c[(starts - 1).clamp_(min=0)], torch.zeros_like(c[starts]))
            z |= ((c - before.repeat_interleave(lengths)) & 1) << bit
            del c, before
        return z
    wide = x.double() if x.dtype.is_floating_point else x.long()
    del x
    if op == "scan":
        return torch.cumsum(wide, 0)
    f = f.clone()
    f[0] = 1
    starts = torch.nonzero(f).view(-1)
    if op == "segsum":
        sums = _sums_between(wide, torch.cat([starts[1:], torch.tensor([wide.numel()], device="cuda")]))
        return _padded(sums, case), torch.tensor([starts.numel()], dtype=torch.int64, device="cuda")
    c = torch.cumsum(wide, 0)
    before = torch.where(starts > 0, c[(starts - 1).clamp_(min=0)], torch.zeros_like(c[starts]))
    del wide
    return c - before.repeat_interleave(torch.diff(starts, append=torch.tensor([c.numel()], device="cuda")))


def tolerance(case):
    """Four times the largest error seen in 32 bits with the row scans made in two orders (the two variants):
    running sums whose carries add up over thousands of tiles 7.4e-7, sums and products of rows 2.2e-7."""
    op = case["op"]
    if op == "compress" or case.get("dtype") in ("i8", "u8"):
        return "exact"
    return {"rel": 3e-6 if op in ("segscan", "scan") else 1e-6}
