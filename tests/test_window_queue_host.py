"""The queue of large windows of the window build, on the host: the rule that says how many entries a window is
queued in (csrc/window_queue.hpp, the header the kernels include) against the room the workspace has for them."""
import os
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

DRIVER = r"""
#include <cstdio>
#include "window_queue.hpp"
int main()  // per line: entries, windows, then (edges of a window, how many windows have them) ... 0
{
    int nnz, n_windows, cnt, times;
    while (std::scanf("%d %d", &nnz, &n_windows) == 2) {
        long long queued = 0;
        while (std::scanf("%d", &cnt) == 1 && cnt > 0) {
            if (std::scanf("%d", &times) != 1) return 1;
            if (cnt > ftc::MID_CAP) queued += static_cast<long long>(times) * ftc::direct_parts(cnt);
        }
        std::printf("%lld %d\n", queued, ftc::direct_capacity(nnz, n_windows));
    }
    return 0;
}
"""


def shapes():
    """Graphs as (nodes, rows per window, {edges of a window: number of such windows})."""
    for n in (16, 64, 700, 2200, 4096, 8192, 9216, 16_384, 46_000):
        for blk_h in (1, 5, 16, 64):                          # complete graphs
            yield n, blk_h, {min(blk_h, n) * n: n // blk_h or 1}
    for cnt in (4097, 8192, 16_384, 32_768, 32_769, 49_153, 70_000, 262_144, 262_145, 600_000, 10 ** 6, 2 ** 31 - 1):
        yield 16, 16, {cnt: 1}                                # one window (repeated columns are legal)
        yield 1, 1, {cnt: 1}
    for n, deg, blk_h in ((16_384, 9000, 16), (8192, 2458, 64), (20_000, 512, 16), (200_000, 2000, 16), (262_144, 8000, 16)):
        yield n, blk_h, {deg * blk_h: n // blk_h}
    rng = np.random.default_rng(0)
    for _ in range(300):                                      # a few sizes mixed
        blk_h = int(rng.integers(1, 65))
        sizes = np.exp(rng.uniform(0, np.log(2_000_000), size=rng.integers(1, 6))).astype(int)
        yield 64 * 1000, blk_h, {int(s): int(rng.integers(1, 50)) for s in sizes}


def test_the_queue_holds_every_part_of_every_window(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("no g++")
    src, exe = tmp_path / "queue.cpp", tmp_path / "queue"
    src.write_text(DRIVER)
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", "-I" + os.path.join(ROOT, "paper_2412_12218_amd", "csrc"),
                    "-o", str(exe), str(src)], check=True)
    lines = []
    for n, blk_h, windows in shapes():
        nnz = sum(c * t for c, t in windows.items())
        if nnz < 2 ** 31:
            lines.append(f"{nnz} {sum(windows.values())} " + " ".join(f"{c} {t}" for c, t in windows.items() if c) + " 0")
    out = subprocess.run([str(exe)], input="\n".join(lines), capture_output=True, text=True, check=True).stdout.split("\n")
    assert len(out) == len(lines) + 1
    for line, got in zip(lines, out):
        queued, room = map(int, got.split())
        assert queued <= room, line
