"""Spinor planes in LDS are written and read as 16-byte vectors (Planes), while
an array of R2<float> is only aligned to 8 bytes: every shared array of R2<R>,
or struct of them, has to ask for 16."""
import glob
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2602_20516_amd", "csrc")


def test_shared_spinor_planes_are_16_byte_aligned():
    n = 0
    for path in sorted(glob.glob(os.path.join(CSRC, "*.h*"))):
        with open(path) as f:
            src = f.read()
        for decl in re.findall(r"__shared__[^;]*;", src):
            name = re.search(r"__shared__\s+(?:__align__\(\d+\)\s+)?(\w+)<R>", decl)
            if not name:
                continue
            n += 1
            own = re.search(rf"struct alignas\(16\) {name.group(1)}\b", src)
            assert "__align__(16)" in decl or own, f"{os.path.basename(path)}: {decl}"
    assert n >= 2
