"""The rules that choose between 32-bit counts and 64-bit sums in the data-derived histogram, evaluated on the host."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SRC = r"""
#include <cstdio>
#include "sop_kparams.h"
int main()
{
    for (unsigned words = 64; words <= SOP_K_DD_MAXBINS; words *= 2)
        for (unsigned wpl = 8; wpl <= 16; wpl += 8)
            for (int flags = 0; flags < 4; ++flags)
                for (long long steps = 1; steps <= 64; steps += 7) {
                    const unsigned n = dd_replicas(words, wpl, flags & 1, flags & 2, steps * 4096, 4096);
                    std::printf("%u %u %d %lld %u %u\n", words, wpl, flags, steps, n, n ? dd_dear_mass(words, wpl, n) : 0u);
                }
}
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    d = tmp_path_factory.mktemp("rules")
    src, exe = d / "r.cpp", d / "r"
    src.write_text(SRC)
    subprocess.check_call(["g++", "-std=c++17", "-I", os.path.join(ROOT, "paper_2605_14929_amd", "csrc"), "-o", str(exe), str(src)])
    out = subprocess.run([str(exe)], capture_output=True, text=True, check=True).stdout
    return [tuple(int(v) for v in line.split()) for line in out.splitlines()]


def test_replicas_fit_and_are_shared_evenly(rules):
    for words, wpl, flags, steps, n, dear in rules:
        assert n in (0, 1, 2, 4, 8, 16)
        assert words * 8 + n * words * 4 <= 136 << 10                  # of 160 KiB, beside the static part


def test_no_replicas_for_few_steps_levels_or_heavy_uniform_norms(rules):
    for words, wpl, flags, steps, n, dear in rules:
        if steps < 8 or flags & 1:
            assert n == 0
        if flags & 2 and n:
            assert (64 * wpl << 20) <= dear


def test_emptying_is_repaid(rules):
    # between two emptyings (words / 64 exchanges and adds a lane) a wavefront under the limit saves at least their cost
    for words, wpl, flags, steps, n, dear in rules:
        if n:
            budget = (2 ** 32 - 1) // (16 // n)
            assert (budget // max(dear, 1) + 1) * wpl * 64 >= 4 * words
