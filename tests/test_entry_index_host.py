"""Entry numbers near INT32_MAX, on the host: batches of entries (csrc/entry_index.hpp, the header the kernels include) stay inside
their range and reach each of its entries once."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

DRIVER = r"""
#include <cstdio>
#include "entry_index.hpp"
int main()  // first, end, places of a batch -> smallest and largest entry that is read, number of entries in the range that were reached
{
    int first, end, batch;
    while (std::scanf("%d %d %d", &first, &end, &batch) == 3) {
        long long lo = 1ll << 40, hi = -(1ll << 40), reached = 0, batches = 0;
        for (uint32_t e0 = first; ftc::entry_in(e0, end) && batches < 100000; e0 += batch, ++batches)
            for (int k = 0; k < batch; ++k) {
                const long long e = ftc::entry_or_last(e0 + k, end);
                lo = e < lo ? e : lo;
                hi = e > hi ? e : hi;
                reached += ftc::entry_in(e0 + k, end);
            }
        std::printf("%lld %lld %lld\n", lo, hi, reached);
    }
    return 0;
}
"""


def test_batches_at_the_end_of_the_largest_graphs(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("no g++")
    src, exe = tmp_path / "entries.cpp", tmp_path / "entries"
    src.write_text(DRIVER)
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", "-fsanitize=undefined", "-fno-sanitize-recover=all",
                    "-I" + os.path.join(ROOT, "paper_2412_12218_amd", "csrc"), "-o", str(exe), str(src)], check=True)
    most = 2 ** 31 - 1
    cases = [(first, end, batch) for end in (1, 511, 512, 513, 4096, most - 512, most - 511, most - 1, most)
             for first in (end - 1, end - 64, end - 3001) if first >= 0 for batch in (512, 1024, 8192)]
    out = subprocess.run([str(exe)], input="\n".join("%d %d %d" % c for c in cases), capture_output=True, text=True, check=True).stdout.split("\n")
    assert len(out) == len(cases) + 1
    for (first, end, _), line in zip(cases, out):
        assert tuple(map(int, line.split())) == (first, end - 1, end - first)
