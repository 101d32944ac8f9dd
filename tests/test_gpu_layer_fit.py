"""The per-layer procedure fits its codebooks on the GPU: candidates, dropped ones among them, their ACos and the winner's table are those of the single
calls chained, with the fits on the host (sop_dd_fit), bit for bit: smallest and largest histograms and codebooks, no rounds and many, pools that are empty or
the whole layer, equal pools, one plane and several passes over the weights."""
import numpy as np
import pytest

import paper_2605_14929_amd as sop
from paper_2605_14929_amd import layer_search
from oracle import atoms as OA
import sop_inputs as si

pytestmark = pytest.mark.gpu

NF, SH = OA.to_f32(OA.nf(4)), OA.to_f32(OA.sh(4))
ATOMS = [NF, SH, OA.to_f32(OA.negate(OA.nf(4))), OA.to_f32(OA.negate(OA.sh(4)))]


@pytest.mark.parametrize("M,K,g", [(48, 1024, 16), (4, 48, 16), (36, 1056, 32)])
@pytest.mark.parametrize("bins,entries,iters,p", [(64, 16, 20, (50.0, 80.0)), (1024, 16, 20, (0.0, 50.0, 70.0, 70.0, 100.0)), (8192, 16, 40, (60.0,)), (2048, 2, 5, (30.0, 60.0, 90.0)),
                                                  (1024, 64, 20, (20.0, 75.0)), (256, 33, 1, (50.0, 95.0)), (512, 16, 0, (40.0,))])
@pytest.mark.parametrize("weighted", [True, False])
def test_against_fits_on_the_host(M, K, g, bins, entries, iters, p, weighted):
    import torch
    W, c = si.bf16_round(si.student_t_weights(M, K, 4.0, 8300 + M)), si.channel_norms(K, 1.0, 8301)
    Wt, ct = torch.from_numpy(W).cuda().to(torch.bfloat16), torch.from_numpy(c).cuda()
    fmt, Nb = sop.fmt_by_name("UE4M3"), M * K // g
    init = NF if entries == 16 else np.linspace(-1, 1, entries, dtype=np.float32)
    cx = sop.Context(0)
    r = layer_search.search_layer(cx, Wt, ct, g, fmt, ATOMS, p_grid=p, fit_entries=entries, fit_iters=iters, fit_bins=bins, fit_init=init, weighted_fit=weighted)
    tops = [int(np.floor(x * Nb / 100.0 + 0.5)) for x in p]
    cx.set_alphabet(ATOMS)
    rank = cx.pair_search(Wt, ct, g, fmt, emit=True).blk_rank
    want, tables = {}, {}
    for a, tab in enumerate(ATOMS):
        level, _, _ = cx.partition_levels(rank[a].clone(), tops)
        hist = cx.dd_histogram_levels(Wt, ct if weighted else None, g, level, len(tops), bins).cpu().numpy()
        js, books = [], []
        for j in range(len(p)):
            if not hist[j].any():
                book = init
            else:
                try:
                    book = sop.sop_dd_fit(hist[j], entries, iters, init)
                except sop.SopError:
                    continue
            js.append(j)
            books.append(np.asarray(book, np.float32))
        if not js:
            continue
        try:
            cx.set_alphabet([tab] + books)
        except sop.SopError:
            continue                                                  # (searched one by one: not followed here)
        cx.set_pairs([(0, 1 + i) for i in range(len(js))])
        acos = cx.pair_search(Wt, ct, g, fmt).acos_pair.cpu().numpy()
        for i, j in enumerate(js):
            want[(a, p[j])] = acos[i]                                 # (equal p: the last one, as the result's dictionary)
            tables.setdefault((a, p[j]), books[i])
    assert {k: v for k, v in r.acos_fitted.items() if k in want} == want
    if r.kind == "fitted":
        assert np.array_equal(r.table_b, tables[(r.a, r.p_percent)])


def test_a_captured_call_is_refused_and_the_graph_stays_good():
    """A refused call, with good arguments or with bad ones, adds nothing to the graph being captured, and the context serves the next call."""
    import torch
    W, c = si.bf16_round(si.student_t_weights(48, 1024, 4.0, 8310)), si.channel_norms(1024, 1.0, 8311)
    Wt, ct = torch.from_numpy(W).cuda().to(torch.bfloat16), torch.from_numpy(c).cuda()
    cx, x = sop.Context(0), torch.zeros(64, device="cuda")
    call = lambda k=0: layer_search.search_layer(cx, Wt, ct, 16, sop.fmt_by_name("UE4M3"), ATOMS, p_grid=(50.0, 80.0), k=k)
    want = call()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        x.add_(1.0)
        for k in (0, 100):                                           # (100: out of range, otherwise found by the first search)
            with pytest.raises(sop.SopError):
                call(k)
        x.add_(1.0)
    for i in range(3):
        graph.replay()
        torch.cuda.synchronize()
        assert (x == 2.0 * (i + 1)).all()
        got = call()
        assert got.acos == want.acos and got.acos_fitted == want.acos_fitted


@pytest.mark.parametrize("bins", [64, 1024, 8192])
def test_fits_that_64_bits_may_not_hold_are_left_to_the_host(bins):
    """The fitting kernel on histograms at the edges of its range: a total mass of 2^62 / bins is fitted, to the host's bits; one more, bins that wrap the total
    to something small or to nothing, and negative ones are not."""
    import ctypes as C
    import torch

    class FitParams(C.Structure):
        _fields_ = [("hist", C.c_void_p), ("n_bins", C.c_int), ("n_entries", C.c_int), ("iters", C.c_int), ("init", C.c_float * 64), ("out", C.c_void_p), ("status", C.c_void_p)]

    OK, EMPTY, HOST = 0, 2, 3
    most = ((1 << 63) - 1 >> 1) // bins
    x = (2.0 * np.arange(bins) + 1.0) / bins - 1.0
    bell = np.floor(np.exp(-4.0 * x * x) / np.exp(-4.0 * x * x).sum() * most * 0.999).astype(np.int64)
    full, over, small, nothing, negative, empty, right = [bell.copy() for _ in range(7)]
    full[bins // 2] += most - int(full.sum())
    over[bins // 2] += most + 1 - int(over.sum())
    small[:] = np.maximum(bell >> 20, 1)
    small[[1, 5, bins - 9, bins - 2]] = 1 << 62                       # (the total is 2^64 and a little)
    nothing[:] = 0
    nothing[[3, bins - 7]] = -(1 << 63)
    negative[bins // 3] = -1
    empty[:] = 0
    right[:bins // 2] = 0
    hist = np.stack([full, over, small, nothing, negative, empty, right])
    want = [OK, HOST, HOST, HOST, HOST, EMPTY, OK]
    entries = 16
    t = torch.from_numpy(hist).cuda()
    out, status = torch.zeros((len(want), 64), device="cuda"), torch.full((len(want),), -1, dtype=torch.int32, device="cuda")
    p = FitParams(t.data_ptr(), bins, entries, 20, (C.c_float * 64)(*NF), out.data_ptr(), status.data_ptr())
    launch = sop.lib().sopk_fit_launch
    launch.argtypes = [C.POINTER(FitParams), C.c_int, C.c_void_p]
    assert launch(C.byref(p), len(want), torch.cuda.current_stream().cuda_stream) == 0
    torch.cuda.synchronize()
    assert status.tolist() == want
    for i in (0, 6):
        assert np.array_equal(out[i, :entries].cpu().numpy(), np.asarray(sop.sop_dd_fit(hist[i], entries, 20, NF), np.float32))


@pytest.mark.parametrize("M,bins,p", [(512, 8192, (20.0,)), (1024, 4096, (20.0, 95.0))])
def test_fits_left_to_the_host_within_the_procedure(M, bins, p, monkeypatch):
    """Norms so small that every weight has the largest mass there is: the first pool's total exceeds what the kernel fits (the second's of the last case does not),
    and its histogram comes to the host."""
    import torch
    K = 1024
    norms = np.full(K, 1e-36, np.float32)
    Wt = torch.from_numpy(si.bf16_round(si.student_t_weights(M, K, 4.0, 8300 + M))).cuda().to(torch.bfloat16)
    total = int(sop.Context(0).dd_histogram(Wt, torch.from_numpy(norms).cuda(), 16, bins).cpu().numpy().sum())
    most = (1 << 62) // bins
    assert [total * (100 - x) / 100 > most for x in p] == [x < 50 for x in p]
    monkeypatch.setattr(si, "channel_norms", lambda *a: norms)
    test_against_fits_on_the_host(M, K, 16, bins, 16, 20, p, True)
