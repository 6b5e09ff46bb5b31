"""The digits after which the selection may end a window early: the source's bound
is where key_after_digit (paper_2607_01757_amd/csrc/lk_key.h) still lies above
every key that shares the leading bits, found here by building it for the host."""
import os
import re
import subprocess

from test_key_after_cpu import CSRC, DRIVER


def test_bound_of_early_window_ends(tmp_path):
    src, exe = tmp_path / "d.cpp", str(tmp_path / "d")
    src.write_text(DRIVER)
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-I" + CSRC, str(src), "-o", exe], check=True)
    keys = [0, 1, 0x7FF0_0000_0000_0000_0000_0000 - 1, 0x3FF1_2345_6789_ABCD_FFFF_FFF0, 0x4000_0000_0000_0000_0000_00FF]
    text = "".join("%x %x %d\n" % (k >> 32, k & 0xFFFFFFFF, p) for p in range(96) for k in keys)
    out = iter(subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout.split("\n"))
    above = {}
    for p in range(96):
        low = max(0, 96 - p - 8)               # key bits below the digit
        got = [int("".join(next(out).split()), 16) for _ in keys]
        above[p] = all(g == ((k >> low) + 1) << low for g, k in zip(got, keys))
    last = max(p for p in above if all(above[i] for i in range(p + 1)))
    text = open(os.path.join(CSRC, "lk_gftt.hip")).read()
    rule = [line for line in text[:text.index("key_after_digit(prefix, d)")].split("\n") if line.strip().startswith("if (")][-1]
    bound = re.search(r"d <= (\d+) &&", rule)
    assert bound and int(bound.group(1)) <= last, (rule, last)
