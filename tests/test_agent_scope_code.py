"""What the compiler makes of the two hand-overs between workgroups that are
ordered by waiting, not by a fence at agent scope (which would write back and
invalidate an XCD's whole L2): the piece sums of a split segment (k_backward_rows:
store, wait, count; who counts last loads all) and the published head counts of
the segment build (k_segments). In the assembly for gfx950, the store has to go
through to where every XCD sees it (sc1), a wait for it has to come before the
count, and the loads have to read from there (sc1), after the count is known."""
import os
import re
import subprocess

import pytest

from paper_2010_13100_amd import build


def functions(source, tmp_path, name):
    """The instructions of the device functions whose name contains `name`."""
    out = os.path.join(tmp_path, "k.s")
    flags = [f for f in build.FLAGS if f not in ("-fPIC", "-Wall")]
    r = subprocess.run([build.HIPCC, *flags, "-w", "--cuda-device-only", "-S",
                        os.path.join(build.CSRC, source), "-o", out], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-1000:]
    with open(out) as f:
        text = f.read()
    got = {m.group(1): re.findall(r"^\t([a-z]\w+[^\n;]*)", m.group(2), re.M)
           for m in re.finditer(r"^(_Z\w*):.*?\n(.*?)^\.Lfunc_end", text, re.M | re.S)
           if name in m.group(1)}
    assert got, name
    return got


def first(code, at, pattern):
    for i in range(at, len(code)):
        if re.search(pattern, code[i]):
            return i
    pytest.fail(f"no {pattern}")


pytestmark = pytest.mark.skipif(not os.path.exists(build.HIPCC), reason="no HIP compiler")
STORE, LOAD = r"^global_store_dword\b.*\bsc1\b", r"^global_load_dword\b.*\bsc1\b"
WAIT = r"^s_waitcnt\b.*vmcnt\(0\)"


def test_piece_sums(tmp_path):
    for name, code in functions("tc_backward.hip", tmp_path, "k_backward_rows").items():
        stores = [i for i, c in enumerate(code) if re.search(STORE, c)]
        loads = [i for i, c in enumerate(code) if re.search(LOAD, c)]
        # one piece end, whose last counter loads up to 32 sums at once
        assert len(stores) == 1 and len(loads) == 32, name
        count = first(code, stores[0], r"^global_atomic_add\b.*\bsc0\b")
        assert first(code, stores[0], WAIT) < count, name
        assert first(code, count, WAIT) < loads[0] and count < loads[0], name


def test_published_head_counts(tmp_path):
    (name, code), = functions("tc_cast.hip", tmp_path, "k_segments").items()
    stores = [c for c in code if re.search(STORE, c)]
    loads = [c for c in code if re.search(LOAD, c)]
    assert len(stores) == 1 and len(loads) >= 1, name
