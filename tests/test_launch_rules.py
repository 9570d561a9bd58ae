"""Rules of the host side that no call can force on a machine at hand, checked on the CPU: those of the C++ side at compile
time (the translation unit is parsed for the host only, with static assertions behind it)."""
import os
import subprocess
import types

import pytest
import torch

from paper_2506_23906_amd import binding, build

CSRC = os.path.dirname(build.SRC)


def holds(tmp_path, condition):
    src = tmp_path / "rule.hip"
    src.write_text('#include "%s"\nstatic_assert(%s, "rule");\n' % (build.SRC, condition))
    flags = [f for f in build.FLAGS if f not in ("-shared", "-fPIC", "-O3", "-Wall")]
    res = subprocess.run([build.HIPCC] + flags + ["--cuda-host-only", "-fsyntax-only", "-w", "-I", CSRC, str(src)],
                         capture_output=True, text=True, timeout=300)
    assert res.returncode == 0 or "static assertion failed" in res.stderr, res.stderr[-2000:]
    return res.returncode == 0


@pytest.mark.parametrize("tiles,resident,first", [(1, 0, 1), (1, 1, 1), (1, 512, 1), (5, 0, 1), (5, 1, 1), (512, 512, 512),
                                                  (513, 512, 512), (4, 512, 4)])
def test_the_first_workgroup_never_draws_a_ticket(tmp_path, tiles, resident, first):
    """resident = 0: the query of how many workgroups the device holds has failed; then one takes the tile of its own index, the
    others tickets."""
    assert holds(tmp_path, "first_round_of(%d, %d) == %d" % (tiles, resident, first))
    assert not holds(tmp_path, "first_round_of(%d, %d) == 0" % (tiles, resident))


def test_the_current_stream_without_the_raw_queries(monkeypatch):
    monkeypatch.setattr(binding, "_raw_stream", None)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: types.SimpleNamespace(cuda_stream=77))
    assert binding._stream_ptr(None) == 77
    assert binding._stream_ptr(types.SimpleNamespace(cuda_stream=5)) == 5
