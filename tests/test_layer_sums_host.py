"""The words of a search's layer sums that count their workgroups, on the host: complete and clear whatever the workgroups add, exact for
every sum a layer can have."""
import os
import subprocess

from test_gpu_layer_sums import ROWS_OF, SETS

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SRC = r"""
#include <cstdio>
#include <cstdint>
#include <initializer_list>
#include <vector>
#include "sop_kparams.h"
// the reduction of one output over g workgroups in the order i * step mod g: true if the last adder sees the count complete, every word is
// clear again and nobody finished before; *total is what it found
static bool reduce(unsigned int g, const std::vector<long long>& v, unsigned int step, long long* total)
{
    unsigned long long row[SOP_K_REPL] = {0};
    int finished = 0;
    for (unsigned int i = 0; i < g; ++i) {
        const unsigned int b = (unsigned int)((unsigned long long)i * step % g), r = b % (SOP_K_REPL - 1), m = sum_members(g, r);
        row[r] += sum_add1(v[b], sum_max(g));
        if ((row[r] >> 56) != m) continue;
        const unsigned long long s = row[r];
        row[r] = 0;
        row[SOP_K_REPL - 1] += sum_add2(s, m);
        if ((row[SOP_K_REPL - 1] >> 60) != sum_rows_used(g)) continue;
        if (i != g - 1 || finished++) return false;
        *total = (long long)(row[SOP_K_REPL - 1] - sum_rows_used(g) * kSumOne2);
        row[SOP_K_REPL - 1] = 0;
    }
    for (unsigned long long w : row) if (w) return false;
    return finished == 1;
}
int main()
{
    for (unsigned int g = 1; g <= SOP_K_SEARCH_MAXWG; ++g) {
        // the largest layer: 2^58 units, spread evenly over 32 or more workgroups (a card's partition has at least 32 compute units)
        const long long most = g >= 32 ? (1ll << 58) / g + (1ll << 30) : 1ll << 40;
        for (unsigned int step : {1u, 257u, 263u}) {             // (primes to every g)
            long long total = 0;
            for (int kind = 0; kind < 6; ++kind) {
                std::vector<long long> v(g);
                long long sum = 0;
                for (unsigned int b = 0; b < g; ++b) {
                    const unsigned long long h = (b + 1) * 0x9E3779B97F4A7C15ull;
                    v[b] = kind == 0 ? 0 : kind == 1 ? most : kind == 2 ? -(long long)(h >> 34) : (long long)(h % (unsigned long long)most);
                    // sums out of a layer's range: of either sign, in some or all of the workgroups
                    if (kind == 4) v[b] = h & (1ull << 40) ? INT64_MIN : -(1ll << 41);
                    if (kind == 5) v[b] = h & (1ull << 40) ? INT64_MAX : -(1ll << 55);
                    if (kind < 4) sum += v[b];
                }
                if (!reduce(g, v, step, &total)) { std::printf("count lost: %u workgroups, kind %d\n", g, kind); return 1; }
                if (kind < 4 && total != sum) { std::printf("sum wrong: %u workgroups, kind %d\n", g, kind); return 1; }
            }
        }
    }
    std::puts("ok");
}
"""


def _build(tmp_path, text):
    src, exe = tmp_path / "s.cpp", tmp_path / "s"
    src.write_text(text)
    subprocess.check_call(["g++", "-std=c++17", "-fsanitize=undefined", "-fno-sanitize-recover", "-I", os.path.join(ROOT, "paper_2605_14929_amd", "csrc"), "-o", str(exe), str(src)])
    return str(exe)


def test_words_complete_and_clear_for_every_sum(tmp_path):
    r = subprocess.run([_build(tmp_path, SRC)], capture_output=True, text=True)
    assert r.stdout.strip() == "ok", r.stdout + r.stderr


def test_the_rows_of_the_gpu_test_take_the_workgroups_it_names(tmp_path):
    """A step a row (rows of 64 lanes are not folded: a fold wastes no fewer lanes than none), 256 compute units, one evaluation a codebook."""
    asked = [(w, M, len(tabs)) for w, M in ROWS_OF.items() for tabs in SETS]
    calls = "".join(f'std::printf("%lld\\n", search_workgroups({M}, 256, {e}));' for _, M, e in asked)
    out = subprocess.run([_build(tmp_path, '#include <cstdio>\n#include "sop_kparams.h"\nint main() { ' + calls + " }")], capture_output=True, text=True, check=True).stdout
    assert [int(x) for x in out.split()] == [w for w, _, _ in asked]
    words = 7                                                         # (first-row words: the grids below, at and above one and two workgroups a word)
    assert {words - 1, words, words + 1, 2 * words - 1, 2 * words, 2 * words + 1} <= set(ROWS_OF)
