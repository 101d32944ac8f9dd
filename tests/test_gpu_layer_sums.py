"""The layer's sums count the workgroups that have added to them: few workgroups, as many as there are words to add to (seven) and one
more or less, twice as many, all of a card's; consecutive calls of different alphabets leave nothing behind."""
import numpy as np
import pytest

import paper_2605_14929_amd as sop
from oracle import atoms as OA, pairsearch as ops
import sop_inputs as si
from gpu_util import compare, oracle_fmt, run_gpu

pytestmark = pytest.mark.gpu

NF, SH = OA.to_f32(OA.nf(4)), OA.to_f32(OA.sh(4))
SETS = [[NF], [NF, SH, OA.to_f32(OA.negate(OA.nf(4)))], [OA.to_f32(OA.nf(5)), NF, SH, OA.to_f32(OA.sh(5)), OA.to_f32(OA.negate(OA.sh(4))), OA.to_f32(OA.negate(OA.nf(4))), OA.to_f32(OA.negate(OA.nf(5)))]]


def leaves_nothing_behind(W, c, g, fmt):
    first = None
    for tabs in SETS + SETS[:1]:
        got = run_gpu(W, c, tabs, g, fmt, emit=False)
        compare(got, ops.pair_search(W, c, tabs, g, oracle_fmt(fmt)), len(tabs) * (len(tabs) - 1) // 2, emit=False)
        if first is None:
            first = got
    assert np.array_equal(got["acos_atom"], first["acos_atom"])       # (the last call repeats the first, bit for bit)


@pytest.mark.parametrize("M", [1, 3, 5, 23, 25, 28, 29, 33, 57, 257, 1023])     # (three steps a row, even numbers of rows folded)
def test_few_to_many_workgroups(M):
    K, g, fmt = 1032, 8, sop.fmt_by_name("UE4M4")                    # 129 lanes: two full strips and one of a single lane
    W, c = si.student_t_weights(M, K, 4.0, 7300 + M), si.channel_norms(K, 1.0, 7301)
    W[0, :512] = 0.0                                                  # blocks without norm count 1
    leaves_nothing_behind(W, c, g, fmt)


# workgroups -> rows of one step each: four steps a workgroup, one step more makes another one
ROWS_OF = {w: 4 * w - (w & 1) for w in (1, 2, 5, 6, 7, 8, 9, 13, 14, 15, 20, 21, 22)}


@pytest.mark.parametrize("workgroups", ROWS_OF)
def test_around_the_number_of_words(workgroups):
    """(That the launch rule gives these rows so many workgroups: test_layer_sums_host.py.)"""
    M, K, g, fmt = ROWS_OF[workgroups], 512, 8, sop.fmt_by_name("UE4M4")     # 64 lanes: a step a row
    W, c = si.student_t_weights(M, K, 4.0, 7600 + M), si.channel_norms(K, 1.0, 7601)
    leaves_nothing_behind(W, c, g, fmt)


def test_a_layer_beyond_binary32_spoils_only_its_own_result():
    """Finite weights whose norms overflow give a NaN deficit, which takes 2^28 a step off a workgroup's sum (the lanes' 32-bit sums wrap): 5120 steps of it
    go below -2^40.  The call that follows is as if there had been none."""
    import torch
    cx = sop.Context(0)                                               # (a context of its own)
    fmt, g = sop.fmt_by_name("UE4M4"), 8
    W, c = si.student_t_weights(64, 1032, 4.0, 7400), si.channel_norms(1032, 1.0, 7401)
    ref = ops.pair_search(W, c, SETS[1], g, oracle_fmt(fmt))
    Wt, ct = torch.from_numpy(W).cuda(), torch.from_numpy(c).cuda()
    cx.set_alphabet(SETS[1])
    big = torch.full((32768, 20480), 1e30, dtype=torch.bfloat16, device="cuda")
    cb = torch.full((20480,), 1e10, dtype=torch.float32, device="cuda")
    cx.pair_search(big, cb, g, fmt, emit=False)
    for _ in range(2):
        out = cx.pair_search(Wt, ct, g, fmt, emit=False)
        assert np.max(np.abs(out.acos_atom.cpu().numpy() - ref.acos_atom)) <= 1e-6
        assert np.max(np.abs(out.acos_pair.cpu().numpy()[:3] - ref.acos_pair)) <= 1e-6
