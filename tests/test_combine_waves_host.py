"""Waves per token of the combine (compiled for the CPU with g++): never more than a launch may have threads, at the largest
batch and beyond any width that fits the card, one per piece of 512 columns wherever that is allowed."""
import os
import subprocess
import tempfile

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = r'''
#include <cstdio>
#include <cstdlib>
#include <cstdint>
#define LORA_HD inline
#include "lora_layout.h"
int main(int argc, char** argv) { for (int i = 1; i + 1 < argc; i += 2) printf("%d\n", lora::combine_waves(atoi(argv[i]), atoi(argv[i + 1]))); return 0; }
'''


@pytest.fixture(scope="module")
def exe():
    d = tempfile.mkdtemp()
    src, out = os.path.join(d, "waves_probe.cpp"), os.path.join(d, "waves_probe")
    open(src, "w").write(SRC)
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-I", os.path.join(ROOT, "paper_2604_07173_amd", "csrc"), src, "-o", out])
    return out


def test_the_launch_stays_within_the_thread_limit(exe):
    cases = [(t, h) for t in (1, 63, 1024, 24577, (1 << 19) + 1, 1 << 20) for h in (8, 512, 520, 4096, 4104, 14336, 40960, 1 << 17, 1 << 24)]
    out = subprocess.check_output([exe, *[str(v) for c in cases for v in c]]).decode().split()
    for (tokens, h), waves in zip(cases, map(int, out)):
        pieces = -(-h // 512)
        assert 1 <= waves <= pieces
        assert -(-tokens * waves // 4) * 256 < 1 << 32, (tokens, h, waves)       # workgroups of 256 threads
        if tokens * pieces <= 24576 or (pieces <= 8 and tokens * pieces < 1 << 25):
            assert waves == pieces, (tokens, h, waves)
