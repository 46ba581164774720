"""Launches over up to eight matrices have a small descriptor table, larger ones the big one: the same kernels, so nine matrices in
one call give what they give in calls of eight and one (which the other tests hold to the oracle)."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2102_08124_amd import binding as tm   # noqa: E402


@pytest.mark.parametrize("dtype,N,M,odd", [(torch.float32, 2, 4, 0), (torch.float32, 4, 8, 0), (torch.float32, 8, 16, 0), (torch.bfloat16, 2, 4, 0),
                                           (torch.bfloat16, 2, 4, 4), (torch.bfloat16, 4, 8, 0), (torch.bfloat16, 8, 16, 0), (torch.float32, 1, 4, 0)])
@pytest.mark.parametrize("fmt", [tm.TMASK_MASK_U8, tm.TMASK_MASK_BITS])
def test_nine_matrices_are_eight_and_one(dtype, N, M, odd, fmt):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(100 * N + M)
    if odd and fmt == tm.TMASK_MASK_BITS:
        pytest.skip("bit masks need widths that are multiples of eight")
    ws = [torch.randn((64 + 16 * k, 128 + 64 * (k % 3) + odd), device="cuda", generator=gen).to(dtype) for k in range(9)]
    wsp = tm.alloc_workspace(ws, N, M)
    res = []
    for groups in ([ws], [ws[:8], ws[8:]]):
        out = []
        for part in groups:
            masks, obj = tm.alloc_masks(part, fmt), torch.zeros(len(part), dtype=torch.float64, device="cuda")
            best, bobj = tm.alloc_masks(part, fmt), torch.zeros(len(part), dtype=torch.float64, device="cuda")
            dense = [torch.zeros_like(w) for w in part]
            score = torch.zeros(len(part) * tm.SCORE_OUT_BYTES, dtype=torch.uint8, device="cuda")
            per = torch.zeros(sum(w.numel() for w in part) // (M * M), device="cuda")
            packed = [tm.alloc_packed(w, N, M) for w in part]
            tm.tmask_approx(part, masks, N, M, objective=obj, mask_fmt=fmt, workspace=wsp)
            tm.tmask_exact(part, best, N, M, objective=bobj, mask_fmt=fmt, workspace=wsp)
            tm.tmask_approx_dense(part, None, dense, N, M, mask_fmt=fmt)
            tm.tmask_score(part, best, N, M, score, per_block_obj=per, mask_fmt=fmt, workspace=wsp)
            tm.tmask_apply_pack(part, best, packed, N, M, mask_fmt=fmt, workspace=wsp)
            torch.cuda.synchronize()
            out.append((masks, best, dense, [obj], [bobj], [score], [per], [t for p in packed for t in p]))
        res.append([[t for o in out for t in o[k]] for k in range(8)])
    for a, b in zip(*res):
        a = torch.cat([t.contiguous().view(-1).view(torch.uint8) for t in a])
        b = torch.cat([t.contiguous().view(-1).view(torch.uint8) for t in b])
        assert torch.equal(a, b)
