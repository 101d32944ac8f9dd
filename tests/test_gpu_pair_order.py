"""The pair stage and the bin records at their edges: every number of atoms in orders that the kernel regroups, ties everywhere (the same codebook twice), part
of the pairs in any order, errors beyond binary32; alphabets whose atoms are evaluated one by one, together, and with the largest tables."""
import itertools

import numpy as np
import pytest

import paper_2605_14929_amd as sop
from oracle import atoms as OA, pairsearch as ops
import sop_inputs as si
from gpu_util import compare, ctx, oracle_fmt, run_gpu

pytestmark = pytest.mark.gpu

NF, SH, NF5, SH5 = (OA.to_f32(t) for t in (OA.nf(4), OA.sh(4), OA.nf(5), OA.sh(5)))
NEG = lambda t: OA.to_f32(-np.asarray(t, dtype=np.float64)[::-1])
# copies before and after their originals, a codebook twice, groups mixed: the internal order swaps many pairs
LONG = [SH, NF, NEG(NF5), NF, NEG(SH), NF5, NEG(NF), SH5]


def _layer(M, K, seed, bf16=False):
    W, c = si.student_t_weights(M, K, 4.0, seed), si.channel_norms(K, 1.0, seed + 1)
    if bf16:
        W = si.generate.bf16_round(W)
    W[1, :64] = 0.0                                               # every atom ties
    c[64:96] = 0.0                                                # errors are zero: every atom ties
    return W, c


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("g", [8, 16, 32])
@pytest.mark.parametrize("fmt,rule", [("UE4M4", 0), ("E4M3", 0), ("E4M3", 1)])
@pytest.mark.parametrize("A", range(2, 9))
def test_ties_and_swapped_pairs(A, fmt, rule, g, bf16):
    W, c = _layer(9, 1120, 8100 + A, bf16)
    fmt = sop.fmt_by_name(fmt)
    for tabs in (LONG[:A], LONG[:A][::-1]):
        got = run_gpu(W, c, tabs, g, fmt, scale_rule=rule, bf16=bf16, emit=False)
        compare(got, ops.pair_search(W, c, tabs, g, oracle_fmt(fmt), scale_rule=rule), A * (A - 1) // 2, emit=False)


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("metric", [sop.SEL_WSE, sop.SEL_MSE, sop.SEL_COS])
@pytest.mark.parametrize("A", [3, 6, 7, 8])
def test_part_of_the_pairs_in_any_order(A, metric, bf16):
    W, c = _layer(6, 1120, 8200 + A, bf16)
    fmt, tabs, rng = sop.fmt_by_name("UE4M4"), LONG[:A], np.random.default_rng(A)
    pairs = list(itertools.combinations(range(A), 2))
    for n in (1, 2, len(pairs) // 2, len(pairs)):
        some = [pairs[i] for i in rng.permutation(len(pairs))[:n]]
        got = run_gpu(W, c, tabs, 16, fmt, metric=metric, pairs=some, bf16=bf16, emit=False)
        compare(got, ops.pair_search(W, c, tabs, 16, oracle_fmt(fmt), metric=metric, pairs=some), n, emit=False)


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("A", [3, 6, 8])
def test_selectors_of_several_layers(A, bf16):
    """The model-wide call: layers of several shapes with selector words and without, ties, copies in the internal order and part of the pairs in an order of
    their own; each layer as in a search of its own, and as the oracle has it."""
    import torch
    fmt, tabs, rng = sop.fmt_by_name("UE4M4"), LONG[:A][::-1], np.random.default_rng(A)
    pairs = list(itertools.combinations(range(A), 2))
    some = [pairs[i] for i in rng.permutation(len(pairs))[:max(2, len(pairs) * 2 // 3)]]
    data = [_layer(M, K, 8600 + i, bf16) for i, (M, K) in enumerate([(9, 1120), (3, 2048), (33, 160), (8, 1120)])]
    cx = ctx()
    cx.set_alphabet(tabs)
    cx.set_pairs(some)
    dt = torch.bfloat16 if bf16 else torch.float32
    layers = [(torch.from_numpy(W).cuda().to(dt), torch.from_numpy(c).cuda()) for W, c in data]
    wide = len(some) > 16
    for want_sel in (True, False):
        acos, atoms, words = cx.pair_search_layers(layers, 16, fmt, want_sel=want_sel)
        torch.cuda.synchronize()
        for i, (W, c) in enumerate(data):
            ref = ops.pair_search(W, c, tabs, 16, oracle_fmt(fmt), pairs=some)
            assert np.max(np.abs(acos[i].cpu().numpy() - ref.acos_pair)) <= 1e-6 and np.max(np.abs(atoms[i].cpu().numpy() - ref.acos_atom)) <= 1e-6
            if want_sel:
                got = words[i].cpu().numpy()
                assert np.array_equal(got.view(np.uint16 if got.dtype == np.int16 else np.uint32).astype(np.uint32).reshape(-1), ref.sel_words)


def test_errors_beyond_binary32_tie():
    """Errors of +infinity are equal; the blocks beside them are not touched."""
    W, c = _layer(8, 512, 8300)
    W[3:5] *= np.float32(1e25)
    fmt = sop.fmt_by_name("UE4M4")
    got, ref = run_gpu(W, c, LONG[:6], 16, fmt, emit=False), ops.pair_search(W, c, LONG[:6], 16, oracle_fmt(fmt))
    assert np.array_equal(got["sel_words"], ref.sel_words)


def _fine(n, step, seed):
    """n entries from -1 to 1, the last but one three boundaries `step` apart: the finer the step, the more bins"""
    t = np.sort(np.random.default_rng(seed).uniform(-0.9, 0.9, n - 5))
    t = t[np.concatenate([[True], np.diff(t) > 2 * step])]
    return np.concatenate([[-1.0], t, 0.93 + step * np.arange(3), [1.0]]).astype(np.float32)


def _alphabet(steps, least_bins, scale):
    """Three codebooks of a table of least_bins at least (the number hangs on where the boundaries fall between the bins as well)"""
    for step in steps:
        tabs = [OA.to_f32(_fine(n, step, seed) * f) for n, seed, f in zip((14, 13, 40), (1, 2, 3), scale)]
        try:
            if sop.sop_check_alphabet(tabs)[0] >= least_bins:
                return tabs
        except sop.SopError:
            break                                                 # (closer than any table resolves)
    raise AssertionError("no such table")


@pytest.mark.parametrize("emit", [False, True])
@pytest.mark.parametrize("steps,least_bins", [((0.02,), 64), (np.arange(0.0031, 0.0008, -2e-5), 1024)])
@pytest.mark.parametrize("scale", [(1.0, 1.0, 1.0), (1.0, 0.96, 0.91)])
def test_bin_records(scale, steps, least_bins, emit):
    """Records of atoms together and of atoms one by one, tables up to the largest, with as many scale codes as are tabulated (the largest of both do not
    fit into LDS where planes are written: the scales are computed)."""
    tabs = _alphabet(steps, least_bins, scale)
    fmt = sop.ScaleFmt(0, 4, 7, 12, -1, -1)                        # 2048 codes
    W, c = _layer(8, 1120, 8400)
    compare(run_gpu(W, c, tabs, 16, fmt, emit=emit), ops.pair_search(W, c, tabs, 16, oracle_fmt(fmt)), 3, emit=emit)


@pytest.mark.parametrize("g", [8, 16, 32])
@pytest.mark.parametrize("fmt,rule", [("UE4M4", 0), ("E4M3", 0), ("E4M3", 1)])
@pytest.mark.parametrize("A", [3, 6, 8])
def test_errors_below_zero_and_errors_that_are_no_numbers(A, fmt, rule, g):
    """Norms that the interface rules out and nothing checks: the errors are compared as numbers all the same (below zero where a norm is), whatever the
    pairs' order, and the blocks beside them are not touched.  A NaN beats nothing and loses to nothing: the block stays with the atom that comes
    first inside the kernel, which a block of nothing but NaNs tells for every pair."""
    W, c = _layer(9, 1120, 8500 + A)
    c[128:640] *= np.where(np.random.default_rng(A).random(512) < 0.3, -1.0, 1.0).astype(np.float32)
    c[704] = np.nan
    c[832] = np.inf
    W[::2, 832] = 0.0                                             # (infinity times a residual of zero)
    fmt = sop.fmt_by_name(fmt)
    pairs = list(itertools.combinations(range(A), 2))
    swapped = 0
    for tabs in (LONG[:A], LONG[:A][::-1]):
        for some in (pairs, pairs[::-1], pairs[1::3]):
            got = run_gpu(W, c, tabs, g, fmt, pairs=some, scale_rule=rule, emit=False)["sel_words"]
            ref = ops.pair_search(W, c, tabs, g, oracle_fmt(fmt), pairs=some, scale_rule=rule)
            first = got[704 // g]
            swapped |= int(first)
            want = ref.sel_words.copy()
            for q, (a, b) in enumerate(some):
                nan = np.isnan(ref.blk_err[a]) | np.isnan(ref.blk_err[b])
                assert nan[704 // g] and nan.sum() >= 9
                want[nan] = want[nan] & ~np.uint32(1 << q) | first & np.uint32(1 << q)
            assert np.array_equal(got, want)
    assert A == 3 or swapped
