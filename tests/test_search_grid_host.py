"""The number of workgroups of a search, evaluated on the host."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SRC = r"""
#include <cstdio>
#include <initializer_list>
#include "sop_kparams.h"
int main()
{
    for (int n_cu : {1, 38, 256})
        for (int w = 1; w <= 4; ++w)
            for (int e = 1; e < 4; ++e)
                for (long long steps = 1; steps < 40000; steps += steps < 5000 ? 1 : 997)
                    std::printf("%d %d %d %lld %lld\n", n_cu, w, e, steps, search_workgroups(steps, n_cu, w, e));
    std::printf("256 4 3 %lld %lld\n", (1ll << 31) - 1, search_workgroups((1ll << 31) - 1, 256, 4, 3));
}
"""


@pytest.fixture(scope="module")
def grid(tmp_path_factory):
    d = tmp_path_factory.mktemp("grid")
    src, exe = d / "g.cpp", d / "g"
    src.write_text(SRC)
    subprocess.check_call(["g++", "-std=c++17", "-I", os.path.join(ROOT, "paper_2605_14929_amd", "csrc"), "-o", str(exe), str(src)])
    out = subprocess.run([str(exe)], capture_output=True, text=True, check=True).stdout
    return [tuple(int(v) for v in line.split()) for line in out.splitlines()]


def _most(steps, wg):
    """Largest number of steps of a SIMD: the kernel cuts [0, steps) evenly over the workgroups and each part over four SIMDs."""
    part = -(-steps // wg)
    return -(-part // 4)


def test_grid_is_within_the_device(grid):
    for n_cu, w, evals, steps, wg in grid:
        assert 1 <= wg <= n_cu


def test_steps_per_simd(grid):
    for n_cu, w, evals, steps, wg in grid:
        best = _most(steps, n_cu)
        if w == 1 and evals > 1 or best > 8 or best == 1 and (evals > 1 or wg == -(-steps // 4)):
            assert _most(steps, wg) == best                   # as few as the device allows
        else:
            assert _most(steps, wg) <= max(best, 5 if evals <= 2 else 3)
