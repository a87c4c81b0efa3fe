"""The counting of positions in rounds (pk_internal.h), up to the longest call that is taken: every position once, none past
the end, no signed 32-bit overflow.  On the host, as the kernels that walk positions use the same code."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdio>
#include "pk_internal.h"
template <int N> bool covers(int64_t n)
{
    int64_t next = 0;                                      // positions counted so far, in 64 bits
    for (pk::Rounds<N> at((int)n); at.any(); at.next()) {
        if ((int64_t)at.base != next || (int64_t)at.left != n - next) return false;
        next += at.left < N ? at.left : N;
        if (next > n) return false;
    }
    return next == n;
}
int main()
{
    const int64_t ns[] = {0, 1, 511, 512, 513, 16384, 16385, (int64_t(1) << 31) - 16384, (int64_t(1) << 31) - 16383, pk::kNnzMax - 1, pk::kNnzMax};
    for (int64_t n : ns)
        if (!covers<512>(n) || !covers<8192>(n) || !covers<16384>(n) || !covers<65536>(n)) { std::printf("%lld\n", (long long)n); return 1; }
    return 0;
}
"""


@pytest.mark.parametrize("flags", [["-O0", "-ftrapv"], ["-O2"]])
def test_rounds_cover_every_position(tmp_path, flags):
    src, exe = tmp_path / "rounds.cpp", tmp_path / "rounds"
    src.write_text(PROGRAM)
    subprocess.check_call(["g++", "-std=c++17", *flags, "-I", os.path.join(ROOT, "include"),
                           "-I", os.path.join(ROOT, "paper_2204_04903_amd", "csrc"), str(src), "-o", str(exe)])
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
