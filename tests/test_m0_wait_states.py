"""Loads straight into LDS in the assembly that this tree's backward kernels compile to.  They take their LDS address from M0, and have to stand
at least one wait state behind the scalar instruction that wrote it: a load that came earlier would put its data elsewhere in LDS, which
no result shows reliably."""
import os
import re
import subprocess

import pytest

from paper_2605_24058_amd import binding

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


def _too_early(lines):
    """Lines of loads into LDS with no wait state between them and the last write of M0 before them."""
    found, since = [], 1   # wait states since M0 was written
    loads = 0
    for n, line in enumerate(lines):
        text = line.split(";")[0].strip()
        if not text or text.startswith(".") or text.endswith(":"):
            continue
        if re.match(r"(global|buffer)_load_\w*lds\w*\s|buffer_load_\w+ .*\blds\b", text):
            loads += 1
            if since < 1:
                found.append(n)
        nop = re.match(r"s_nop (\d+)", text)
        if re.match(r"s_\w+ m0\b", text):
            since = 0
        else:
            since += int(nop.group(1)) + 1 if nop else 1
    return found, loads


def test_what_counts_as_too_early():
    load = "\tglobal_load_lds_dwordx4 v[2:3], off nt"
    assert _too_early(["\ts_mov_b32 m0, s3", load])[0] == [1]
    assert _too_early(["\ts_add_i32 m0, s3, s4", "\t;;#ASMSTART", load])[0] == [2]
    assert _too_early(["\ts_mov_b32 m0, s3", "\ts_nop 0", load])[0] == []
    assert _too_early(["\ts_mov_b32 m0, s3", "\tv_mov_b32_e32 v1, v2", load, "\ts_mov_b32 m0, s4", load])[0] == [4]


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="needs hipcc")
def test_loads_into_lds_wait_for_m0(tmp_path):
    out = str(tmp_path / "lordba_backward.s")
    flags = [f for f in binding.HIPCC_FLAGS if f != "-shared"]
    subprocess.run([HIPCC] + flags + ["-I", os.path.join(binding._ROOT, "include"), "--cuda-device-only", "-S",
                                      os.path.join(binding._CSRC, "lordba_backward.hip"), "-o", out], check=True, capture_output=True, timeout=300)
    with open(out) as f:
        early, loads = _too_early(f.read().splitlines())
    assert loads > 0
    assert early == []
