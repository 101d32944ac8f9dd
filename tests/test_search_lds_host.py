"""What a search keeps in LDS, evaluated on the host: the table of scales stays there for every alphabet, scale word and plane but the largest."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LDS = 160 * 1024

SRC = r"""
#include <cstddef>
#include <cstdio>
#include <initializer_list>
#include "sop_kparams.h"
int main()
{
    for (int na : {2, 6, 8})
        for (int rec : {SOP_K_BIN_BYTES, SOP_K_PAIR_BIN_BYTES, SOP_K_WIDE_BIN_BYTES(na)})
            for (int bins : {16, 40, 512, 768, 1024})
                for (int codes : {15, 256, 1200, 2047, 2048})
                    for (bool cosine : {false, true}) {
                        const int kept = search_tab_codes(na, cosine, bins, rec, codes, 160 * 1024);
                        std::printf("%d %d %d %d %d %zu %d %zu\n", na, rec == SOP_K_WIDE_BIN_BYTES(na), bins, codes, kept, search_lds(na, cosine, bins, rec, kept),
                                    cosine, search_lds(na, cosine, bins, rec, 0) - bins * rec);
                    }
}
"""


@pytest.fixture(scope="module")
def table(tmp_path_factory):
    d = tmp_path_factory.mktemp("lds")
    src, exe = d / "l.cpp", d / "l"
    src.write_text(SRC)
    subprocess.check_call(["g++", "-std=c++17", "-I", os.path.join(ROOT, "paper_2605_14929_amd", "csrc"), "-o", str(exe), str(src)])
    out = subprocess.run([str(exe)], capture_output=True, text=True, check=True).stdout
    return [tuple(int(v) for v in line.split()) for line in out.splitlines()]


def test_scales_are_tabulated_wherever_they_fit(table):
    for na, planes, bins, codes, kept, lds, cosine, rest in table:
        assert lds + 1024 <= LDS
        assert kept == (0 if planes and na == 8 and bins == 1024 and codes > 1200 else codes), (na, planes, bins, codes)


def test_selector_tables_only_where_pairs_are_chained(table):
    """All that is left beside bins and scales: below 1 KiB (group parameters, outputs, sums), and a KiB per eight pairs of a chain."""
    for na, planes, bins, codes, kept, lds, cosine, rest in table:
        assert rest // 1024 == (0 if cosine else {2: 0, 6: 2, 8: 4}[na])
