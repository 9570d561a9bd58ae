"""The binding's calls through the extension that marshals their arguments, and what it leaves to the lines in Python."""
import os
import sys
import types

import numpy as np
import pytest
import torch

from paper_2506_23906_amd import binding as B
from paper_2506_23906_amd import build
from paper_2506_23906_amd import workloads as W


def test_what_it_does_not_know_is_left_to_python(libmmvseg_path):
    B.load()
    m, t = B._marshal, torch.zeros(64)
    f = torch.zeros(64, dtype=torch.uint8)
    for z, ws in ((t, f), (None, f), (t, None)):               # CPU tensors, arguments left out
        assert m.segscan(t, f, None, z, "mfma", ws, None) is None
    assert m.scan(t, 3.0, t, "mfma", f, None) is None and m.scan(t, 3, t, "other", f, None) is None
    assert m.compress(None, f, 64, t, t, f, None) is None
    assert m.spmv_csr(8, 8, None, t, t, t, t, t, "mfma", f, None) is None
    with pytest.raises(TypeError):
        m.segscan(t, f)
    with pytest.raises(TypeError):
        m.bind(1)
    with pytest.raises(B.MmvError):                            # ... which raises what it raised before
        B.mmv_segscan(t, f, z=t, ws=f)


@pytest.mark.parametrize("module", [None, types.SimpleNamespace(torch_version="another")])   # not built; built for another torch
def test_the_library_loads_without_the_extension(libmmvseg_path, monkeypatch, tmp_path, module):
    monkeypatch.setitem(sys.modules, B.__package__ + "._marshal", module)
    monkeypatch.delattr(sys.modules[B.__package__], "_marshal", raising=False)
    monkeypatch.setattr(B, "MARSHAL_PATH", str(tmp_path / "_marshal.so"))
    monkeypatch.setattr(B, "_lib", None)
    monkeypatch.setattr(B, "_marshal", None)
    assert B.load().mmv_status_string(0) and B._marshal is None
    with pytest.raises(B.MmvError):
        B.mmv_segscan(torch.zeros(64), torch.zeros(64, dtype=torch.uint8))


def test_a_failed_compilation_replaces_nothing(monkeypatch, tmp_path):
    def run(cmd, **_):
        made = cmd[cmd.index("-o") + 1]
        assert os.path.dirname(made) == str(tmp_path)
        open(made, "w").write("new")
        return types.SimpleNamespace(returncode=1 if cmd[0] == "g++" else 0, stderr="")
    for name in ("LIB", "MARSHAL_LIB"):
        (tmp_path / name).write_text("old")
        monkeypatch.setattr(build, name, str(tmp_path / name))
    monkeypatch.setattr(build, "subprocess", types.SimpleNamespace(run=run))
    with pytest.raises(RuntimeError):
        build.build()
    assert (tmp_path / "LIB").read_text() == (tmp_path / "MARSHAL_LIB").read_text() == "old"


@pytest.mark.gpu
def test_both_ways_give_the_same(monkeypatch):
    n = 5000
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    rng = np.random.default_rng(3)
    row, col, val, xv = W.spmv_coo_zipf(700, 600, 9000, cap=300, seed=5)
    rowptr, f = dev(W.csr_rowptr(row, 700)), dev((rng.random(n) < 0.1).astype(np.uint8))
    row, col, val, xv = dev(row), dev(col), dev(val), dev(xv)
    bits = dev(W.pack_flags(f.cpu().numpy()).view(np.int32))
    x = dev(rng.integers(-3, 4, size=n).astype(np.float32))
    side = torch.cuda.Stream()

    def calls(how):
        kept = []   # every tensor until the end: a kernel on another stream may still use it, and its memory goes to the next one made
        def keep(tensor):
            kept.append(tensor)
            return tensor
        new = lambda k, dt=torch.float32: keep(torch.zeros(k, dtype=dt, device="cuda"))
        scratch = lambda *a: keep(B.new_workspace(*a))
        out = []
        def call(entry, *a, **kw):
            side.wait_stream(torch.cuda.current_stream())      # (behind the fills)
            r = entry(*a, **kw, **how)
            out.extend(r if isinstance(r, tuple) else [r])
        for xt in (x, x.half(), x.bfloat16(), x.to(torch.int8), x.to(torch.int8).view(torch.uint8)):
            dt = B._DTYPES[keep(xt).dtype]
            for fl in (f, bits):
                ff = B._flag_fmt(fl)
                call(B.mmv_segscan, xt, fl, n=n, z=new(n, B._OUT_DTYPE[dt]), ws=scratch(B.MMV_OP_SEGSCAN, dt, ff, n))
                call(B.mmv_segsum, xt, fl, out=new(n, B._OUT_DTYPE[dt]), nseg=new(1, torch.int64), variant="shuffle",
                     ws=scratch(B.MMV_OP_SEGSUM, dt, ff, n), n=n)
            call(B.mmv_scan, xt, n=n - 7, z=new(n, B._OUT_DTYPE[dt]), ws=scratch(B.MMV_OP_SCAN, dt, 1, n))
        for v in (x, None):
            call(B.mmv_compress, v, f, n, out=new(n, torch.float32 if v is not None else torch.int32), count=new(1, torch.int64),
                 ws=scratch(B.MMV_OP_COMPRESS, B.MMV_I8_I32, 0, n))
        coo = lambda: scratch(B.MMV_OP_SPMV_COO, B.MMV_F32_F32, B.MMV_FLAGS_PACKED32, val.numel())
        csr = lambda: keep(B.workspace(B.mmv_spmv_csr_workspace_bytes(700, val.numel())))
        call(B.mmv_spmv_coo, 700, 600, row, col, val, xv, y=new(700), ws=coo())
        ws = coo()
        call(B.mmv_spmv_coo_prepare, 700, 600, row, col, ws=ws)
        out.pop()                                              # (the plan)
        call(B.mmv_spmv_coo_run, 700, 600, row, col, val, xv, ws, y=new(700))
        call(B.mmv_spmv_csr, 700, 600, rowptr, col, val, xv, y=new(700), ws=csr())
        ws = csr()
        call(B.mmv_spmv_csr_prepare, 700, 600, rowptr, col, ws=ws)
        out.pop()
        call(B.mmv_spmv_csr_run, 700, 600, rowptr, col, val, xv, ws, y=new(700))
        torch.cuda.synchronize()
        return out

    here = calls({})
    with torch.cuda.stream(side):
        there = calls({})
    named = calls({"stream": side})
    monkeypatch.setattr(B, "_marshal", None)
    python = calls({})
    assert len(here) == len(python) == len(named) == len(there)
    for a, b, c, d in zip(here, python, named, there):
        assert torch.equal(a, b) and torch.equal(c, b) and torch.equal(d, b)
