"""The ranking counts [7/8, 1) finer than the rest in its first pass: thresholds inside it, outside it and in both at once, scores at its
ends, all in one bin, infinities and NaN, against a sort of the keys; calls of one and of several planes' worth of thresholds in turn leave nothing behind."""
import numpy as np
import pytest

import paper_2605_14929_amd as sop

pytestmark = pytest.mark.gpu


def keys(s, higher):
    u = np.where(s == 0, np.float32(0), s).astype(np.float32).view(np.uint32)
    k = np.where(u >> 31 != 0, ~u, u | np.uint32(0x80000000))
    return k if higher else ~k


def scores(kind, n, rng):
    half, below_one = np.float32(0.875), np.nextafter(np.float32(1), np.float32(0))
    if kind == "inside":
        return (1.0 - np.abs(rng.standard_normal(n)) * 0.02).clip(0.875, below_one).astype(np.float32)
    if kind == "ends":
        e = np.array([half, np.nextafter(half, np.float32(0)), np.nextafter(half, np.float32(1)), below_one, 1.0, np.nextafter(np.float32(1), np.float32(2)), 0.9375, -0.875, -0.9375, -1.0], np.float32)
        return e[rng.integers(0, len(e), n)]
    if kind == "wide":
        return (np.exp(rng.standard_normal(n) * 8) * rng.choice([-1, 1], n)).astype(np.float32)
    if kind == "both":
        return np.where(rng.random(n) < 0.5, 1.0 - rng.random(n) * 0.4, rng.standard_normal(n) * 3).astype(np.float32)
    if kind == "one bin":
        return (np.float32(0.9375).view(np.uint32) + rng.integers(0, 256, n).astype(np.uint32)).view(np.float32)
    s = rng.standard_normal(n).astype(np.float32)
    s[::5], s[1::7], s[2::11], s[3::13], s[4::17] = np.inf, -np.inf, np.nan, -0.0, 0.75
    return s


@pytest.mark.parametrize("kind", ["inside", "ends", "wide", "both", "one bin", "special"])
@pytest.mark.parametrize("higher", [True, False])
def test_against_sorted_keys(kind, higher):
    import torch
    rng = np.random.default_rng(5)
    cx = sop.Context(0)
    for n in (1, 7, 4096, 70003, 600000) + ((9_000_003,) if kind in ("inside", "both") else ()):
        s = scores(kind, n, rng)
        k = keys(s, higher)
        order = np.sort(k)[::-1]
        t = torch.from_numpy(s).cuda()
        for tops in ([n // 2], sorted({0, 1, n // 3, n // 2, n // 2 + 1, n - n // 9, n}), [0], [(n + 1) // 2, n]):
            level, tau, n_a = [x.cpu().numpy() for x in cx.partition_levels(t, tops, higher)]
            want = np.zeros(n, np.int64)
            for j, top in enumerate(tops):
                if top == 0:
                    want += 1
                    assert n_a[j] == 0 and tau[j] == (np.inf if higher else -np.inf)
                    continue
                thr = order[top - 1]
                want += k < thr
                assert n_a[j] == np.count_nonzero(k >= thr), (n, tops, j)
                assert keys(tau[j:j + 1], higher)[0] == thr, (n, tops, j)
            assert np.array_equal(level, want), (n, tops)
        pool, tau, n_a = [x.cpu().numpy() for x in cx.partition(t, (n + 1) // 2, higher)]
        thr = order[(n + 1) // 2 - 1]
        assert np.array_equal(pool, k < thr) and n_a[0] == np.count_nonzero(k >= thr)


def test_replays_of_a_captured_call():
    """A call leaves its counts at zero itself: a graph of one ranking gives the same again and again, with new scores and with other calls between."""
    import torch
    rng = np.random.default_rng(6)
    cx = sop.Context(0)
    for n, tops in ((70004, [100, 35002, 60000]), (9_000_003, [4_500_001])):
        t = torch.from_numpy(scores("both", n, rng)).cuda()
        cx.partition_levels(t, tops)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            out = cx.partition_levels(t, tops) if len(tops) > 1 else cx.partition(t, tops[0])
        for i in range(4):
            t.copy_(torch.from_numpy(scores("both" if i & 1 else "inside", n, rng)))
            graph.replay()
            torch.cuda.synchronize()
            got = [x.cpu().numpy() for x in out]
            if i == 2:
                cx.partition_levels(t, [5, n])
            want = [x.cpu().numpy() for x in (cx.partition_levels(t, tops) if len(tops) > 1 else cx.partition(t, tops[0]))]
            assert all(np.array_equal(a, b) for a, b in zip(got, want)), (n, i)
            k = np.sort(keys(t.cpu().numpy(), True))[::-1]
            assert [int(v) for v in got[2]] == [int(np.count_nonzero(k >= k[m - 1])) for m in tops], (n, i)


@pytest.mark.parametrize("n", [7, 4099, 70004, 2_818_048])
def test_replays_of_a_captured_call_with_one_threshold(n):
    """The same for the three passes of a single threshold, with other calls of other sizes, and calls without a first pool, between the replays."""
    import torch
    rng = np.random.default_rng(7)
    cx = sop.Context(0)
    top = (n + 1) // 2
    t = torch.from_numpy(scores("both", n, rng)).cuda()
    cx.partition(t, top)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        out = cx.partition(t, top)
    for i in range(5):
        s = scores(("both", "inside", "wide", "one bin", "special")[i], n, rng)
        t.copy_(torch.from_numpy(s))
        graph.replay()
        torch.cuda.synchronize()
        pool, tau, n_a = [x.cpu().numpy() for x in out]
        k = keys(s, True)
        thr = np.sort(k)[::-1][top - 1]
        assert np.array_equal(pool, k < thr) and n_a[0] == np.count_nonzero(k >= thr) and keys(tau, True)[0] == thr, (n, i)
        if i == 1:
            cx.partition(t, 0)
        if i == 2:
            cx.partition(t, n)
            cx.partition(t[:max(n // 3, 1)], 1, False)
