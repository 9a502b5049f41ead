"""The upsampling's thread index at sizes past 2^31 threads (a 512^3 grid with 72 channels; a test
cannot allocate it): the host compiler builds the function that the kernel calls, and its
voxel and channel must be those of exact integers.  CPU only."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_index_past_31_bits(tmp_path):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    cases = []                                   # block, thread, C, n0, n1, n2
    for n0, n1, n2, C in ((512, 512, 512, 72), (512, 512, 512, 112), (1024, 516, 260, 112), (8, 12, 4, 16)):
        total = n0 * n1 * n2 * C // 4
        assert total < 2 ** 32
        for i in (0, 1, C // 4, 2 ** 31 - 1, 2 ** 31, 2 ** 31 + 12345, total - 1, total):
            if i <= total:
                cases.append((i // 256, i % 256, C, n0, n1, n2))
    src = tmp_path / "up2.cpp"
    src.write_text('#include <cstdio>\n#include "up2.hpp"\nint main() {\n' + "".join(
        '{ const auto q = ertvie::up2_cell(%uu, 256u, %uu, %uu, %uu, %uu);'
        ' std::printf("%%u %%u %%u %%u %%u\\n", q.v, q.x, q.y, q.z, q.c); }\n' % c[:5] for c in cases) + "return 0; }\n")
    exe = tmp_path / "up2"
    subprocess.run([cxx, "-std=c++17", "-I", os.path.join(ROOT, "paper_1610_00835_amd", "csrc"), str(src), "-o", str(exe)],
                   check=True)
    out = subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.splitlines()
    assert len(out) == len(cases)
    for line, (block, thread, C, n0, n1, n2) in zip(out, cases):
        v, c = divmod(256 * block + thread, C // 4)
        want = (v, v % n0, v // n0 % n1, v // (n0 * n1), 4 * c)
        assert tuple(map(int, line.split())) == want
        assert (want[3] >= n2) == (256 * block + thread == n0 * n1 * n2 * C // 4)
