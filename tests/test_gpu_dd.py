"""GPU parity of the data-derived codebook: the integer histogram of the HIP path against the
oracle's (bit-exact), the fitted table, and the pair search with the fitted atom appended."""
import numpy as np
import pytest

import paper_2605_14929_amd as sop
from oracle import atoms as OA, dd as DD, pairsearch as ops
import sop_inputs as si
from gpu_util import run_gpu, compare, oracle_fmt, ctx, cached_config

pytestmark = pytest.mark.gpu


def gpu_hist(W, c, g, H, bf16, ldw=None, row_step=1, mask=None):
    import torch
    Wt = torch.from_numpy(W).cuda()
    if bf16:
        Wt = Wt.to(torch.bfloat16)
    if ldw is not None:
        buf = torch.zeros((W.shape[0], ldw), dtype=Wt.dtype, device="cuda")
        buf[:, :W.shape[1]] = Wt
        Wt = buf[:, :W.shape[1]]
    ct = None if c is None else torch.from_numpy(c).cuda()
    mt = None if mask is None else torch.from_numpy(mask).cuda()
    h = ctx().dd_histogram(Wt, ct, g, H, row_step, block_mask=mt)
    torch.cuda.synchronize()
    return h.cpu().numpy()


@pytest.mark.parametrize("g", [8, 16, 32, 64])
@pytest.mark.parametrize("bf16", [False, True])
def test_histogram_block_sizes_dtypes_ragged(g, bf16):
    M, K = 37, 1088                                                   # ragged last strip, uneven row ranges
    W = si.student_t_weights(M, K, 4.0, 900 + g, row_sigma=0.5, outlier_frac=0.002)
    if bf16:
        W = si.bf16_round(W)
    W[3, :] = 0.0                                                     # zero blocks are skipped
    W[5, 64:128] = -np.abs(W[5, 64:128])
    c = si.channel_norms(K, 1.0, 901)
    c[200:216] = 0.0
    for H in (256, 1024):
        assert np.array_equal(gpu_hist(W, c, g, H, bf16), DD.histogram(W, c, g, H))
    assert np.array_equal(gpu_hist(W, None, g, 512, bf16), DD.histogram(W, None, g, 512))
    for step in (2, 5, 64):                                           # a sample of the rows: 0, step, 2*step, ...
        assert np.array_equal(gpu_hist(W, c, g, 256, bf16, row_step=step), DD.histogram(W[::step], c, g, 256))


def test_histogram_row_stride_and_bin_counts():
    M, K = 16, 512
    W = si.student_t_weights(M, K, 4.0, 911)
    c = si.channel_norms(K, 1.0, 912)
    assert np.array_equal(gpu_hist(W, c, 16, 64, False, ldw=K + 64), DD.histogram(W, c, 16, 64))
    assert np.array_equal(gpu_hist(W, c, 16, 8192, False), DD.histogram(W, c, 16, 8192))
    import torch
    with pytest.raises(sop.SopError) as e:
        ctx().dd_histogram(torch.from_numpy(W).cuda(), torch.from_numpy(c).cuda(), 16, 1000)
    assert e.value.status == 1
    with pytest.raises(sop.SopError) as e:
        ctx().dd_histogram(torch.from_numpy(W).cuda(), torch.from_numpy(c).cuda(), 12, 1024)
    assert e.value.status == 2


def test_histogram_is_reproducible_and_full_layer():
    W, c, cfg = cached_config("C3_down")
    a = gpu_hist(W, c, 16, 1024, True)
    b = gpu_hist(W, c, 16, 1024, True)
    assert np.array_equal(a, b)
    assert np.array_equal(a, DD.histogram(W, c, 16, 1024))


def test_dd4_joins_the_alphabet_config5_shape():
    # 70B-shaped MLP layer 28672 x 8192: histogram and fit on the whole layer, then the seven-atom
    # search (21 pairs, 32-bit selector words) against the oracle on the whole layer
    W, c, cfg = cached_config("C5")
    g, H = 16, 4096
    hist = gpu_hist(W, c, g, H, True)
    assert np.array_equal(hist, DD.histogram(W, c, g, H))
    init = sop.sop_atom_nf(4)
    dd4 = sop.sop_dd_fit(hist, 16, 20, init)                          # 16 centroids, 20 rounds, from NF4
    assert np.array_equal(dd4, DD.fit(hist, 16, 20, OA.to_f32(OA.nf(4)).astype(np.float64)).astype(np.float32))
    tabs = sop.build_alphabet(cfg["atoms"], bof_draws=si.normal_draws(1 << 20, 4242)) + [dd4]
    fmt = sop.fmt_by_name(cfg["fmt"])
    gpu = run_gpu(W, c, tabs, g, fmt, bf16=True, emit=False)
    ref = ops.pair_search(W, c, tabs, g, oracle_fmt(fmt), want_codes=False)
    compare(gpu, ref, 21, emit=False)
    # the atom fitted to this layer beats every fixed atom on it
    assert gpu["acos_atom"][6] > gpu["acos_atom"][:6].max()
    # a fit from every 16th row is the same grid to within two histogram bins
    h16 = gpu_hist(W, c, g, H, True, row_step=16)
    assert np.array_equal(h16, DD.histogram(W[::16], c, g, H))
    assert np.max(np.abs(sop.sop_dd_fit(h16, 16, 20, init) - dd4)) < 4e-3


@pytest.mark.parametrize("g", [8, 16, 32, 64])
def test_histogram_of_a_pool_of_blocks(g):
    M, K = 41, 1088
    W = si.bf16_round(si.student_t_weights(M, K, 4.0, 950 + g, row_sigma=0.5))
    c = si.channel_norms(K, 1.0, 951)
    rng = np.random.default_rng(952 + g)
    mask = (rng.random(M * K // g) < 0.35).astype(np.uint8)
    mask[mask == 1] = rng.integers(1, 256, int(mask.sum())).astype(np.uint8)      # any non-zero byte counts
    for row_step in (1, 3):
        ref_mask = mask.copy().reshape(M, K // g)
        keep = np.zeros(M, bool); keep[::row_step] = True
        ref_mask[~keep] = 0
        ref = DD.histogram(W, c, g, 512, block_mask=ref_mask.reshape(-1))
        got = gpu_hist(W, c, g, 512, True, row_step=row_step, mask=mask)
        assert np.array_equal(got, ref)
    assert gpu_hist(W, c, g, 512, True, mask=np.zeros_like(mask)).sum() == 0


def test_grid_constrained_dd4_joins_the_alphabet():
    # the codebook selected among the E4M3 grid's values (step 1 of the pair search, data-adaptive atom)
    # from the GPU's histogram: same selection as the oracle's, and as an atom it serves the layer better
    # than the free fit or NF4 snapped to the same grid
    M, K, g, H = 512, 4096, 16, 1024
    W = si.bf16_round(si.student_t_weights(M, K, 4.0, 7300, row_sigma=0.5, outlier_frac=0.001))
    c = si.channel_norms(K, 1.0, 7301)
    hist = gpu_hist(W, c, g, H, True)
    assert np.array_equal(hist, DD.histogram(W, c, g, H))
    grid = sop.sop_weight_grid(sop.WeightFmt(4, 3, -1, -1))
    cand = grid / grid[-1]
    idx, cost = sop.sop_dd_fit_grid(hist, cand, 16)
    ridx, rcost = DD.fit_grid(hist, cand, 16)
    assert abs(cost - rcost) <= 1e-11 * rcost and np.array_equal(idx, ridx)
    dd_grid = cand[idx].astype(np.float32)
    free = sop.sop_dd_fit(hist, 16, 20, sop.sop_atom_nf(4)).astype(np.float64)
    snapped = np.unique(cand[np.abs(cand[None, :] - free[:, None]).argmin(axis=1)]).astype(np.float32)
    nf = sop.sop_atom_nf(4).astype(np.float64)
    nf_snapped = np.unique(cand[np.abs(cand[None, :] - nf[:, None]).argmin(axis=1)]).astype(np.float32)
    assert snapped.size == 16 and nf_snapped.size == 16
    tabs = [sop.sop_atom_nf(4), dd_grid, snapped, nf_snapped]
    fmt = sop.fmt_by_name("UE4M4")
    gpu = run_gpu(W, c, tabs, g, fmt, bf16=True, emit=True)
    ref = ops.pair_search(W, c, tabs, g, oracle_fmt(fmt))
    assert np.array_equal(gpu["sel_words"], ref.sel_words) and np.array_equal(gpu["scale_code"], ref.scale_code)
    for a in range(4):
        assert np.array_equal(gpu["codes"][a], ref.codes[a])
    assert np.max(np.abs(gpu["acos_atom"] - ref.acos_atom)) <= 1e-6
    # among codebooks that live on the E4M3 grid, the one selected on the grid serves the layer best
    # (the unconstrained NF4 table, which no E4M3 LUT can hold, is better still)
    assert gpu["acos_atom"][1] > gpu["acos_atom"][2] and gpu["acos_atom"][1] > gpu["acos_atom"][3]


@pytest.mark.parametrize("H", [64, 1024, 4096, 8192])
@pytest.mark.parametrize("norms", ["ones", "none", "mixed"])
def test_counts_past_32_bits_on_one_bin(H, norms):
    """Every weight of a block at its maximum: whole rows fall on one bin, twelve rows a wavefront, so the 32-bit counts have
    to be emptied on the way (at 8192 bins a single step exceeds the wavefront's share of them).  Expected in closed form."""
    import torch
    M, K, g = 12 * 4096, 1024, 16
    Wt = torch.full((M, K), 0.5, dtype=torch.bfloat16, device="cuda")
    Wt[:, 512:] = -0.25
    c = None if norms == "none" else torch.ones(K, device="cuda")
    if norms == "mixed":
        c[::2] = 0.5
    h = ctx().dd_histogram(Wt, c, g, H).cpu().numpy()
    per_half = M * (512 if norms != "mixed" else 384) << 20
    want = np.zeros(H, dtype=np.int64)
    want[H - 1], want[0] = per_half, per_half
    assert np.array_equal(h, want)


@pytest.mark.parametrize("H,cols", [(64, 1024), (1024, 1024), (2048, 6), (4096, 1024)])
def test_norms_below_the_range_of_the_mass_scale(H, cols):
    """Largest channel norm below 2^20 / FLT_MAX: the scale to integer masses overflows and every non-zero norm counts as the
    largest 32-bit integer.  A step's additions then exceed 32 bits; the sums are exact all the same.  Expected in closed form."""
    import torch
    M, K, g = 12 * 4096, 1024, 16
    Wt = torch.full((M, K), 0.5, dtype=torch.bfloat16, device="cuda")
    Wt[:, 512:] = -0.25
    c = torch.zeros(K, device="cuda")
    c[:cols // 2] = 1e-36
    c[K - cols // 2:] = 1e-36
    h = ctx().dd_histogram(Wt, c, g, H).cpu().numpy()
    want = np.zeros(H, dtype=np.int64)
    want[H - 1] = want[0] = M * (cols // 2) * (2 ** 31 - 1)
    assert np.array_equal(h, want)


@pytest.mark.parametrize("M,K,H", [(12 * 4096, 1024, 1024), (300, 131072, 2048), (300, 131072, 8192)])
def test_strips_of_light_and_heavy_norms(M, K, H):
    """Column masses that differ from strip to strip by four orders of magnitude: a wavefront goes from 32-bit counts to 64-bit
    sums and back.  Expected in closed form: every weight of a block at its maximum."""
    import torch
    g, S = 16, 1024                                                   # a strip: 64 lanes of 16 weights
    Wt = torch.full((M, K), 0.5, dtype=torch.bfloat16, device="cuda")
    Wt[:, ::2 * g] = -0.5
    c = torch.full((K,), 0.75, device="cuda")
    for s in range(0, K, 3 * S):
        c[s:s + S] = 2.0 ** -14
    c[K - 1] = 1.0
    h = ctx().dd_histogram(Wt, c, g, H).cpu().numpy()
    mass = np.rint(c.cpu().numpy().astype(np.float64) * 1048576.0).astype(np.int64)
    want = np.zeros(H, dtype=np.int64)
    want[0] = M * mass[::2 * g].sum()
    want[H - 1] = M * mass.sum() - want[0]
    assert np.array_equal(h, want)


@pytest.mark.parametrize("H", [4096, 8192])
def test_time_does_not_depend_on_the_spread_of_the_norms(H):
    """Norms near their maximum fill the 32-bit counts within a few steps.  Emptying them each time took three times as long as
    the whole pass; the pass now stays within a quarter of its time under widely spread norms (twice is allowed here)."""
    import torch
    W = torch.randn(4096, 11008, device="cuda").to(torch.bfloat16)
    t = {}
    for sigma in (1.0, 0.3, 0.1, 0.0):
        c = (torch.randn(11008, device="cuda") * sigma).exp_()
        for _ in range(3):
            ctx().dd_histogram(W, c, 16, H)
        best = float("inf")
        for _ in range(5):
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            for _ in range(20):
                ctx().dd_histogram(W, c, 16, H)
            e1.record()
            e1.synchronize()
            best = min(best, e0.elapsed_time(e1))
        t[sigma] = best
    assert max(t.values()) < 2.0 * t[1.0], t


@pytest.mark.parametrize("Ms,K", [(129, 1040), (255, 3072), (300, 5024), (1531, 3072), (4097, 16384)])
@pytest.mark.parametrize("form", ["plain", "row_step", "mask", "levels"])
def test_bands_of_rows_with_a_short_last_one(Ms, K, form):
    """Layers of full bands of 128 rows and a shorter one, several strips a row: wavefronts that begin and end anywhere in them,
    with one step each, with several, and (the last size) with enough for 32-bit counts."""
    import torch
    g, H, bf16 = 16, 1024, K != 3072
    step = 3 if form == "row_step" else 1
    M = Ms * step - (step - 1)                                        # Ms sampled rows
    W = si.student_t_weights(M, K, 4.0, 960 + Ms, row_sigma=0.5)
    if bf16:
        W = si.bf16_round(W)
    c = si.channel_norms(K, 1.0, 961)
    rng = np.random.default_rng(962 + Ms)
    if form == "mask":
        mask = (rng.random(M * K // g) < 0.4).astype(np.uint8)
        assert np.array_equal(gpu_hist(W, c, g, H, bf16, mask=mask), DD.histogram(W, c, g, H, block_mask=mask))
    elif form == "levels":
        lv = rng.integers(0, 4, M * K // g).astype(np.uint8)
        Wt = torch.from_numpy(W).cuda()
        h = ctx().dd_histogram_levels(Wt.to(torch.bfloat16) if bf16 else Wt, torch.from_numpy(c).cuda(), g, torch.from_numpy(lv).cuda(), 3, H).cpu().numpy()
        for j in range(3):
            assert np.array_equal(h[j], DD.histogram(W, c, g, H, block_mask=(lv > j).astype(np.uint8)))
    else:
        assert np.array_equal(gpu_hist(W, c, g, H, bf16, row_step=step), DD.histogram(W[::step], c, g, H))


@pytest.mark.parametrize("workgroups", [1, 63, 64, 66, 131, 256])
def test_workgroups_divided_among_rows_of_sums(workgroups):
    """One row of running sums below 64 workgroups or above 1024 words, four otherwise (uneven for 66 and 131); calls of both kinds one
    after the other leave nothing behind.  Integers: equal bit for bit."""
    import torch
    M, K, g = 16 * workgroups - (workgroups > 1), 1024, 16            # a strip a row, 16 rows a workgroup, the last one a row short
    W = si.student_t_weights(M, K, 4.0, 950 + workgroups)
    c = si.channel_norms(K, 1.0, 951)
    level = np.random.default_rng(952).integers(0, 4, M * (K // g)).astype(np.uint8)
    for H in (64, 2048, 1024, 512):
        assert np.array_equal(gpu_hist(W, c, g, H, False), DD.histogram(W, c, g, H))
    for H in (256, 1024):                                             # 768 and 3072 words: no powers of two
        got = ctx().dd_histogram_levels(torch.from_numpy(W).cuda(), torch.from_numpy(c).cuda(), g, torch.from_numpy(level).cuda(), 3, H).cpu().numpy()
        for j in range(3):
            assert np.array_equal(got[j], DD.histogram(W, c, g, H, block_mask=(level > j).astype(np.uint8))), (H, j)
