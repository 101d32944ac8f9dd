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
        for (int e : {1, 2, 6, 16, 32})
            for (long long steps = 1; steps < 40000; steps += steps < 3000 ? 7 : 997)
                std::printf("%d %d %lld %lld\n", n_cu, e, steps, search_workgroups(steps, n_cu, e));
    std::printf("256 6 %lld %lld\n", (1ll << 31) - 1, search_workgroups((1ll << 31) - 1, 256, 6));
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
    for n_cu, evals, steps, wg in grid:
        assert 1 <= wg <= n_cu


def test_grid_is_the_cheapest_of_all(grid):
    for n_cu, evals, steps, wg in grid:
        least = _most(steps, n_cu)
        if least > 8:
            assert wg == n_cu
            continue
        cost = lambda w: 3 * _most(steps, w) * (300 + 100 * evals) + 10 * w      # (thirds of a nanosecond)
        assert cost(wg) <= min(cost(w) for w in range(1, n_cu + 1) if _most(steps, w) <= 8)


def test_wavefronts_of_dear_steps_get_one_each_where_they_can(grid):
    for n_cu, evals, steps, wg in grid:
        if evals >= 16 and steps <= 4 * n_cu:
            assert _most(steps, wg) == 1


FEWER = r"""
#include <cstdio>
#include <initializer_list>
#include "sop_kparams.h"
int main()
{
    long long fewer = 0, bad = 0;
    for (int n_cu : {1, 38, 255, 256})
        for (int e : {1, 2, 6, 12, 24})
            for (long long steps = 1; steps < 9000; ++steps) {
                const long long wg = search_workgroups(steps, n_cu, e);
                const int waves = search_waves(4, steps, wg);
                for (int na : {2, 6, 8}) {
                    if (search_slots(na) / 4 > 4 * waves) ++bad;                       // a wavefront for every four columns of sums in LDS
                    for (bool emit : {false, true}) if (waves != 4) { ++fewer; bad += !search_deal(na, emit, steps, n_cu); }
                }
            }
    std::printf("%lld %lld\n", fewer, bad);
}
"""


def test_a_launch_of_fewer_wavefronts_says_so(tmp_path):
    """The kernel takes its number of threads from KParams::deal, which is 0 where the first steps are not dealt out: never in a launch of fewer wavefronts than
    the variant is built for, or its loops over threads would leave out words."""
    (tmp_path / "f.cpp").write_text(FEWER)
    subprocess.check_call(["g++", "-std=c++17", "-I", os.path.join(ROOT, "paper_2605_14929_amd", "csrc"), "-o", str(tmp_path / "f"), str(tmp_path / "f.cpp")])
    fewer, bad = (int(v) for v in subprocess.run([str(tmp_path / "f")], capture_output=True, text=True, check=True).stdout.split())
    assert fewer > 0 and bad == 0
