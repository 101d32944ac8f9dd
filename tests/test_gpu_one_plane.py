"""Searches that write the ranking scores or the block errors alone have kernels of their own: their planes, selectors and ACos are those of the
call that writes every plane, bit for bit (same integers, same sums).  Sizes: a single block, a strip and one lane more, rows apart in memory, several
steps a wavefront; scale words that saturate (clamped look-ups, direct cosine sums); a copy under a signed word."""
import numpy as np
import pytest

import paper_2605_14929_amd as sop
from oracle import atoms as OA
import sop_inputs as si

pytestmark = pytest.mark.gpu

NF, SH = OA.to_f32(OA.nf(4)), OA.to_f32(OA.sh(4))
NEG, NF5, OWN = OA.to_f32(OA.negate(OA.nf(4))), OA.to_f32(OA.nf(5)), (np.linspace(-1, 1, 16) ** 3 * 0.875).astype(np.float32)
SETS = {1: [NF], 2: [NF, NEG], 3: [NF, SH, OWN], 6: [NF, SH, NEG, OA.to_f32(OA.negate(OA.sh(4))), NF5, OWN]}


@pytest.mark.parametrize("M,K,pad", [(1, 64, 0), (3, 1088, 0), (37, 1024, 8), (700, 4160, 24)])
@pytest.mark.parametrize("g", [8, 16, 32, 64])
@pytest.mark.parametrize("fmt", ["UE4M4", "E4M3", "saturating", "saturating signed"])
@pytest.mark.parametrize("f32", [False, True])
def test_one_plane_against_all(M, K, pad, g, fmt, f32):
    import torch
    W, c = si.student_t_weights(M, K, 3.0, 8100 + M), si.channel_norms(K, 1.0, 8101)
    W[0, :g] = 0.0
    Wt = torch.zeros((M, K + pad), dtype=torch.float32 if f32 else torch.bfloat16, device="cuda")
    Wt[:, :K] = torch.from_numpy(W)
    Wt, ct = Wt[:, :K], torch.from_numpy(c).cuda()
    f = {"saturating": sop.ScaleFmt(0, 2, 3, 0, 1, 20), "saturating signed": sop.ScaleFmt(1, 2, 3, 0, 1, 20)}.get(fmt) or sop.fmt_by_name(fmt)
    Nb = M * (K // g)
    cx = sop.Context(0)
    for A, tabs in SETS.items():
        cx.set_alphabet(tabs)
        full = cx.pair_search(Wt, ct, g, f, emit=True)
        for plane in ("blk_rank", "blk_err"):
            out = sop.Outputs(acos_atom=torch.full((A,), np.nan, dtype=torch.float64, device="cuda"))
            if A > 1:
                out.acos_pair = torch.full((A * (A - 1) // 2,), np.nan, dtype=torch.float64, device="cuda")
                out.sel_words = torch.full((Nb,), -1, dtype=torch.int16, device="cuda")
            buf = torch.full((A * Nb + 64,), -7.0, dtype=torch.float32, device="cuda")          # (64 words behind the planes stay as they are)
            setattr(out, plane, buf[:A * Nb].view(A, Nb))
            cx.pair_search(Wt, ct, g, f, out=out)
            for name in ("acos_atom", "acos_pair", "sel_words"):
                if getattr(out, name) is not None:
                    assert torch.equal(getattr(out, name), getattr(full, name)), (A, plane, name)
            assert torch.equal(buf[:A * Nb].view(A, Nb).view(torch.int32), getattr(full, plane).view(torch.int32)), (A, plane)
            assert bool((buf[A * Nb:] == -7.0).all())
