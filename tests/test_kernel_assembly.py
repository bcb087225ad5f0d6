"""Registers of kernels whose speed rests on how many of their waves a SIMD holds, read from the
assembly that the compiler writes for the repository's own sources (no GPU)."""
import os
import re
import subprocess

import pytest

from paper_1409_6070_amd import build


def kernels(source, tmp_path):
    """{mangled name: (vector registers, scalar registers)} of a source's kernels."""
    out = tmp_path / "k.s"
    cmd = [build.HIPCC, *build.CFLAGS, "-w", "-I", os.path.join(build.HERE, "..", "include"), "--cuda-device-only", "-S",
           os.path.join(build.CSRC, source), "-o", str(out)]
    subprocess.run(cmd, check=True, timeout=300, stdout=subprocess.DEVNULL, stderr=subprocess.DEVNULL)
    got, name, sgpr = {}, None, None
    for line in out.read_text().splitlines():
        m = re.match(r"\s+\.(name|sgpr_count|vgpr_count):\s+(\S+)", line)
        if not m:
            continue
        if m[1] == "name":
            name = m[2]
        elif m[1] == "sgpr_count":
            sgpr = int(m[2])
        else:
            got[name] = (int(m[2]), sgpr)
    return got


def waves_per_simd(vgpr, sgpr):
    """gfx950: 512 vector registers a lane in steps of 8, 800 scalar registers in steps of 16, at most 8 waves."""
    return min(8, 512 // (-(-vgpr // 8) * 8), 800 // (-(-sgpr // 16) * 16))


def test_window_lists_of_32_words_hold_eight_waves(tmp_path):
    got = {n: r for n, r in kernels("rulebook.hip", tmp_path).items() if re.search(r"k_rb_listsILb[01]ELi32E", n)}
    assert len(got) == 2, got
    assert all(waves_per_simd(*r) == 8 for r in got.values()), got
