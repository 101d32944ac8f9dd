"""Atoms of a scale group are evaluated together (four, two or one at a time) and the planes of a search come from one pass:
every grouping, with ordinary blocks beside blocks whose scale saturates (scaled weights beyond the table) or vanishes
(no reconstruction), every set of planes that selects a pass of its own, against the oracle."""
import numpy as np
import pytest

import paper_2605_14929_amd as sop
from oracle import atoms as OA, pairsearch as ops
import sop_inputs as si
from gpu_util import compare, ctx, oracle_fmt, run_gpu

pytestmark = pytest.mark.gpu

M, K = 5, 1088                                   # 68 lanes of 16 weights: a full strip and one of four lanes


def _book(n, lo, hi, seed):
    """n ascending entries from lo to hi, at least a hundredth of the range apart."""
    gaps = np.random.default_rng(seed).uniform(1.0, 2.0, n - 1)
    z = np.concatenate([[0.0], np.cumsum(gaps) / gaps.sum()])
    t = lo + (hi - lo) * z
    t[0], t[-1] = lo, hi
    return OA.to_f32(t)


# atoms per scale group, in order of first appearance (the groups' endpoints differ)
PATTERNS = {"1": [1], "2": [2], "1+1": [1, 1], "1+2": [1, 2], "4": [4], "4+1+1": [4, 1, 1], "3+2": [3, 2], "6": [6], "2+4": [2, 4], "4+3": [4, 3], "8": [8], "1+3+4": [1, 3, 4]}
ENDS = [(-1.0, 1.0), (-1.0, 0.75), (-0.5, 1.0)]


def _tabs(name):
    return [_book(16 if j % 3 else 7, *ENDS[gi], 100 * gi + j) for gi, n in enumerate(PATTERNS[name]) for j in range(n)]


def _weights(bf16, seed):
    W = si.student_t_weights(M, K, 4.0, seed, row_sigma=0.5)
    W[1] *= np.float32(2.0 ** 14)                # saturates the scale word
    W[2, :K // 2] *= np.float32(2.0 ** -16)      # vanishes in it
    W[3, 16:80] = 0.0
    return si.bf16_round(W) if bf16 else W


@pytest.mark.parametrize("name", PATTERNS)
@pytest.mark.parametrize("g,bf16,metric", [(16, True, 0), (16, False, 2), (32, True, 2), (64, False, 0), (8, True, 0)])
def test_every_grouping(name, g, bf16, metric):
    tabs, fmt = _tabs(name), sop.fmt_by_name("UE4M4")
    W, c = _weights(bf16, 31), si.channel_norms(K, 1.0, 32)
    ref = ops.pair_search(W, c, tabs, g, oracle_fmt(fmt), metric=metric, want_codes=True)
    P = len(tabs) * (len(tabs) - 1) // 2
    for emit in (False, True):
        compare(run_gpu(W, c, tabs, g, fmt, metric=metric, bf16=bf16, emit=emit), ref, P, emit=emit)


@pytest.mark.parametrize("planes", [("blk_rank",), ("blk_err",), ("blk_cos", "blk_rank"), ("codes", "scale_code"), ("codes", "blk_rank"), ("blk_err", "blk_cos")])
@pytest.mark.parametrize("name,fmt_name,g", [("2", "UE4M4", 16), ("4+1+1", "UE4M3", 16), ("2", "S1E5M5", 16), ("1+2", "E4M3", 32), ("2", "E4M3", 8)])
def test_every_set_of_planes(planes, name, fmt_name, g):
    import torch
    tabs, fmt = _tabs(name), sop.fmt_by_name(fmt_name)
    W, c = _weights(True, 41), si.channel_norms(K, 1.0, 42)
    ref = ops.pair_search(W, c, tabs, g, oracle_fmt(fmt), want_codes=True)
    cx = ctx()
    cx.set_alphabet(tabs)
    full = cx.alloc_outputs(M, K, g, emit=True)
    for n in ("codes", "scale_code", "blk_cos", "blk_err", "blk_rank"):
        if n not in planes:
            setattr(full, n, None)
    cx.pair_search(torch.from_numpy(W).cuda().to(torch.bfloat16), torch.from_numpy(c).cuda(), g, fmt, out=full)
    torch.cuda.synchronize()
    assert np.array_equal(full.sel_words.cpu().numpy().view(np.uint16).astype(np.uint32), ref.sel_words)
    assert np.abs(full.acos_atom.cpu().numpy() - ref.acos_atom).max() <= 1e-6
    if "blk_rank" in planes:
        assert np.array_equal(full.blk_rank.cpu().numpy().view(np.uint32), ref.blk_rank.view(np.uint32))
    if "blk_err" in planes:
        assert np.array_equal(full.blk_err.cpu().numpy(), ref.blk_err)
    if "blk_cos" in planes:
        assert np.abs(full.blk_cos.cpu().numpy() - ref.blk_cos).max() <= 2e-5       # (the bound of the other parity tests)
    if "scale_code" in planes:
        assert np.array_equal(full.scale_code.cpu().numpy().view(np.uint16), ref.scale_code)
    if "codes" in planes:
        for x, y in zip(full.code_planes, ref.codes):
            assert np.array_equal(x.cpu().numpy(), y)


@pytest.mark.parametrize("name", PATTERNS)
@pytest.mark.parametrize("g,bf16", [(16, True), (16, False), (32, False), (64, True)])
def test_every_grouping_under_the_cosine_metric(name, g, bf16):
    """The searches and the planes of one and two atoms evaluate groups of atoms; wider planes atom by atom.  The model-wide search gives the
    single call's bits."""
    import torch
    tabs, fmt = _tabs(name), sop.fmt_by_name("UE4M4")
    W, c = _weights(bf16, 41), si.channel_norms(K, 1.0, 42)
    ref = ops.pair_search(W, c, tabs, g, oracle_fmt(fmt), metric=1, want_codes=True)
    P = len(tabs) * (len(tabs) - 1) // 2
    for emit in (False, True):
        got = run_gpu(W, c, tabs, g, fmt, metric=1, bf16=bf16, emit=emit)
        compare(got, ref, P, emit=emit)
    Wt = torch.from_numpy(W).cuda()
    pairs, atoms, _ = ctx().pair_search_layers([(Wt.to(torch.bfloat16) if bf16 else Wt, torch.from_numpy(c).cuda())] * 3, g, fmt, metric=1)
    for l in range(3):
        assert np.array_equal(atoms[l].cpu().numpy(), got["acos_atom"])
        if P:
            assert np.array_equal(pairs[l].cpu().numpy(), got["acos_pair"])
