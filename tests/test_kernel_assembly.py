"""What the compiler makes of the repository's own kernels where their speed rests on how many of their
waves a SIMD holds, or their soundness on the order of memory operations: read from the assembly that
it writes for the sources (no GPU)."""
import os
import re
import subprocess

import pytest

from paper_1409_6070_amd import build


def assembly(source, tmp_path):
    out = tmp_path / "k.s"
    cmd = [build.HIPCC, *build.CFLAGS, "-w", "-I", os.path.join(build.HERE, "..", "include"), "--cuda-device-only", "-S",
           os.path.join(build.CSRC, source), "-o", str(out)]
    subprocess.run(cmd, check=True, timeout=300, stdout=subprocess.DEVNULL, stderr=subprocess.DEVNULL)
    return out.read_text().splitlines()


def kernels(source, tmp_path):
    """{mangled name: (vector registers, scalar registers)} of a source's kernels."""
    got, name, sgpr = {}, None, None
    for line in assembly(source, tmp_path):
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


def test_softmax_releases_and_acquires_its_loss_terms(tmp_path):
    """Every workgroup's terms are written back before it raises the counter (buffer_wbl2, waited for), and
    the one that sums them drops what its XCD's caches hold (buffer_inv) before it reads them."""
    lines, seen = assembly("head.hip", tmp_path), 0
    for at, line in enumerate(lines):
        if not re.match(r"_ZN4sscn14k_softmax_xent\S*:", line):
            continue
        end = next(i for i in range(at, len(lines)) if lines[i].strip().startswith(".section"))
        body = [x.split()[0] for x in lines[at:end] if x.startswith("\t") and x.split()]
        add = body.index("global_atomic_add")
        back = [i for i in range(add) if body[i] == "buffer_wbl2"]
        assert back and "s_waitcnt" in body[back[-1]:add], line
        inv = body.index("buffer_inv", add)
        assert "s_barrier" in body[add:inv] and any(x.startswith("global_load") for x in body[inv:]), line
        seen += 1
    assert seen == 2
