"""The rank-key helper that ends a selection window above a digit
(key_after_digit, paper_2607_01757_amd/csrc/lk_key.h), built for the host,
against Python integers."""
import os
import random
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2607_01757_amd", "csrc")

DRIVER = r"""
#define __host__
#define __device__
#define __forceinline__ inline
#include "lk_key.h"
#include <cstdio>
int main()
{
    unsigned long long hi;
    unsigned lo;
    int p;
    while (std::scanf("%llx %x %d", &hi, &lo, &p) == 3) {
        const lkmi::Key k = lkmi::key_after_digit(lkmi::Key{hi, lo}, p);
        std::printf("%016llx %08x\n", k.hi, k.lo);
    }
}
"""


def test_key_after_digit(tmp_path):
    src, exe = tmp_path / "d.cpp", str(tmp_path / "d")
    src.write_text(DRIVER)
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-I" + CSRC, str(src), "-o", exe], check=True)
    rng = random.Random(3)
    cases = []
    for p in list(range(96)) * 40:
        k = rng.getrandbits(96) >> 1                       # R is finite: never all ones
        if rng.random() < 0.4:                             # a run of ones below the digit, a carry through it
            k |= ((1 << rng.randrange(1, 90)) - 1) << rng.randrange(0, 40) & ((1 << 95) - 1)
        cases.append((k, p))
    text = "".join("%x %x %d\n" % (k >> 32, k & 0xFFFFFFFF, p) for k, p in cases)
    out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout.split("\n")
    for (k, p), line in zip(cases, out):
        if p + 8 > 96:                                     # the digit reaches past the key: it names one key
            want = (((k << 32) >> (120 - p)) + 1) << (120 - p) >> 32
        else:
            sh = 96 - p - 8
            want = ((k >> sh) + 1) << sh                   # past every key with these leading p + 8 bits
            assert want > (k | ((1 << sh) - 1)) and want - 1 == (k | ((1 << sh) - 1))
        a, b = line.split()
        assert (int(a, 16) << 32 | int(b, 16)) == want & ((1 << 96) - 1)
