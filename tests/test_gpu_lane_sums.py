"""Searches whose lanes keep their running sums in LDS: the sums are integers, so every pair's ACos equals, bit for bit, what a search of its two
atoms alone (sums in registers) gives: shares long enough for the words to be emptied on the way, shares of seven to nine steps, where a launch
has three or four wavefronts per SIMD, a single step, blocks without norm."""
import os
import subprocess

import numpy as np
import pytest

import paper_2605_14929_amd as sop
from oracle import atoms as OA

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
NF, SH = OA.to_f32(OA.nf(4)), OA.to_f32(OA.sh(4))
OWN = (np.linspace(-1, 1, 16) ** 3 * 0.875).astype(np.float32)       # a codebook with endpoints of its own
SIX = [NF, SH, OA.to_f32(OA.negate(OA.nf(4))), OA.to_f32(OA.negate(OA.sh(4))), OA.to_f32(OA.nf(5)), OWN]
EIGHT = SIX + [OA.to_f32(OA.sh(5)), (np.linspace(-1, 1, 16) * 0.75).astype(np.float32)]


def against_pairs(M, K, g, dtype, tabs, fmt, metric=sop.SEL_WSE, rule=sop.SCALE_ABSMAX, pairs=None):
    import torch
    gen = torch.Generator(device="cuda").manual_seed(M + K)
    W = torch.randn((M, K), generator=gen, device="cuda", dtype=torch.float32).to(dtype)
    c = torch.rand(K, generator=gen, device="cuda") + 0.5
    W[0, :4 * g] = 0                                                 # blocks without norm
    fmt = sop.fmt_by_name(fmt)
    cx = sop.Context(0)
    cx.set_scale_rule(rule)
    A = len(tabs)
    cx.set_alphabet(tabs)
    first = cx.pair_search(W, c, g, fmt, metric=metric)
    again = cx.pair_search(W, c, g, fmt, metric=metric)
    got = {k: getattr(first, k).cpu().numpy() for k in ("acos_pair", "acos_atom", "sel_words")}
    for k in got:
        assert np.array_equal(got[k], getattr(again, k).cpu().numpy()), k
    del again
    sel = got["sel_words"].astype(np.int64)
    q = 0
    for a in range(A):
        for b in range(a + 1, A):
            if pairs is None or (a, b) in pairs:
                cx.set_alphabet([tabs[a], tabs[b]])
                one = cx.pair_search(W, c, g, fmt, metric=metric)
                assert one.acos_pair.cpu().numpy()[0] == got["acos_pair"][q], (a, b)
                assert np.array_equal(one.acos_atom.cpu().numpy(), got["acos_atom"][[a, b]]), (a, b)
                assert np.array_equal(one.sel_words.cpu().numpy().astype(np.int64) & 1, (sel >> q) & 1), (a, b)
            q += 1


# (rows of 5024 columns, g = 32: five steps a row, so seven to nine steps a SIMD of 256 compute units; rows of 1024: a step each)
@pytest.mark.gpu
@pytest.mark.parametrize("rows", [1, 5, 1433, 1480, 1638, 1640])
@pytest.mark.parametrize("tabs,fmt,metric,rule,f32", [
    (SIX, "E4M3", sop.SEL_WSE, sop.SCALE_ABSMAX, False), (SIX, "E4M3", sop.SEL_COS, sop.SCALE_ABSMAX, True), (SIX, "UE4M4", sop.SEL_COS, sop.SCALE_ABSMAX, True),
    (EIGHT, "UE4M4", sop.SEL_WSE, sop.SCALE_ABSMAX, False), (EIGHT, "E4M3", sop.SEL_MSE, sop.SCALE_ABSMAX, False), (EIGHT, "E4M3", sop.SEL_COS, sop.SCALE_ARGMAX, False),
    (SIX, "E4M3", sop.SEL_WSE, sop.SCALE_ARGMAX, True)])
def test_short_and_middling_shares(rows, tabs, fmt, metric, rule, f32):
    import torch
    against_pairs(rows, 5024, 32, torch.float32 if f32 else torch.bfloat16, tabs, fmt, metric, rule, pairs={(0, 1), (1, 5), (2, 3), (0, len(tabs) - 1)})


@pytest.mark.gpu
@pytest.mark.parametrize("rows", [1, 733, 900])                      # (lanes of eight weights: ten steps a row)
@pytest.mark.parametrize("tabs,fmt,metric,rule", [(SIX, "E4M3", sop.SEL_WSE, sop.SCALE_ABSMAX), (EIGHT, "UE4M4", sop.SEL_MSE, sop.SCALE_ABSMAX), (EIGHT, "E4M3", sop.SEL_COS, sop.SCALE_ABSMAX),
                                                  (EIGHT[:7], "E4M3", sop.SEL_WSE, sop.SCALE_ARGMAX)])
def test_lanes_of_eight_weights(rows, tabs, fmt, metric, rule):
    import torch
    against_pairs(rows, 5024, 8, torch.bfloat16, tabs, fmt, metric, rule, pairs={(0, 1), (1, 5), (2, 3), (0, len(tabs) - 1)})


@pytest.mark.gpu
@pytest.mark.parametrize("tabs,fmt", [(EIGHT[:7], "UE4M4"), (SIX, "E4M3")])
def test_words_emptied_on_the_way(tabs, fmt):
    """More than 60 steps a wavefront on 256 compute units: 4 * 256 * 4 * 60 steps of 1024 weights and some."""
    import torch
    against_pairs(33000, 8192, 16, torch.bfloat16, tabs, fmt, pairs={(0, 1), (2, 5)})


SRC = r"""
#include <cstdio>
#include <initializer_list>
#include "sop_kparams.h"
int main()
{
    int bad = 0;
    for (int na : {6, 8})                                  // the largest tables leave room for the sums
        for (int rec : {SOP_K_BIN_BYTES, SOP_K_PAIR_BIN_BYTES})
            for (bool cosine : {false, true})
                bad += search_tab_codes(na, cosine, SOP_K_MAXBINS, rec, SOP_K_MAXTABCODES, 160 * 1024 - lane_sums_bytes(na)) != SOP_K_MAXTABCODES;
    bad += (long long)4 * SOP_K_FLUSH_STEPS << 23 >= 1ll << 31;      // a word's steps
    for (long long steps = 1; steps < 20000; ++steps) {    // wavefronts: as many as built for, but for shares of eight steps
        const long long wg = search_workgroups(steps, 256, 6), most = ((steps + wg - 1) / wg + 3) / 4;
        for (int occ = 1; occ <= 4; ++occ) bad += search_waves(occ, steps, wg) != (occ == 4 && most == 8 ? 3 : occ);
    }
    std::printf("%d\n", bad);
}
"""


def test_room_range_and_wavefronts(tmp_path):
    (tmp_path / "l.cpp").write_text(SRC)
    subprocess.check_call(["g++", "-std=c++17", "-I", os.path.join(ROOT, "paper_2605_14929_amd", "csrc"), "-o", str(tmp_path / "l"), str(tmp_path / "l.cpp")])
    assert subprocess.run([str(tmp_path / "l")], capture_output=True, text=True, check=True).stdout.strip() == "0"
