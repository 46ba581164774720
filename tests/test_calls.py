"""The native half of binding.py takes the usual arguments and leaves every other one to the Python half: it never raises, and on
the GPU both halves give the same outputs and the same errors."""
import types

import pytest

torch = pytest.importorskip("torch")

from paper_2102_08124_amd import binding as tm   # noqa: E402

NONE = types.SimpleNamespace(**{name: (lambda *a: None) for name in ("batch", "dense", "score", "spmm24")})


def test_unusual_arguments_are_left_to_the_python_half():
    L = tm.load_library()
    at, calls = L.at["tmask_approx"], tm._calls
    head = [at, 64, 0, 0, 2, 4, 0]                             # no matrices: refused before the array is read
    t = torch.zeros((4, 64), dtype=torch.bfloat16)
    for k, odd in [(0, 0), (0, None), (1, 0), (1, "x"), (2, 1.0), (3, None), (4, 2 ** 40), (5, -2 ** 31 - 1), (6, t)]:
        args = list(head)
        args[k] = odd
        assert calls.batch(*args, None, 0) is None and calls.dense(*args, 0) is None
        assert calls.score(*args, t, 0, None, None, 0) is None
    for workspace in (7, "x", [], torch.Tensor):
        assert calls.batch(*head, workspace, types.SimpleNamespace(cuda_stream=0)) is None
    for stream in (7, "x", types.SimpleNamespace(cuda_stream="x")):
        assert calls.batch(*head, None, stream) is None
    for short in ([], head):
        assert calls.batch(*short) is None and calls.dense(*short) is None and calls.score(*short) is None and calls.spmm24(*short) is None
    assert calls.batch(*head, None, types.SimpleNamespace(cuda_stream=0)) == tm.TMASK_ERR_SHAPE
    assert calls.spmm24(L.at["tmask_spmm24"], t, t, 4, 64, t, t, None) is None          # no device memory, wrong types


def _outcome(f):
    try:
        f()
        torch.cuda.synchronize()
        return None
    except Exception as e:
        return type(e), str(e)


@pytest.mark.gpu
def test_both_halves_do_the_same(monkeypatch):
    lib, native = tm.load_library(), tm._calls
    w = [torch.randn((256, 128), device="cuda")]
    masks, wsp = tm.alloc_masks(w), tm.alloc_workspace(w, 2, 4)
    obj = torch.zeros(1, dtype=torch.float64, device="cuda")
    batch = tm.MatBatch(w, masks, obj)
    out = torch.zeros(tm.SCORE_OUT_BYTES, dtype=torch.uint8, device="cuda")
    per = torch.zeros(64 * 32, device="cuda")
    dst = [torch.zeros_like(w[0])]
    wb = torch.randn((64, 128), device="cuda").to(torch.bfloat16)
    vals, idx = tm.alloc_packed(wb, 2, 4)[:2]
    vals.copy_(torch.randn(vals.shape, device="cuda"))
    idx.fill_(0x44)
    x, y = torch.randn((8, 128), device="cuda").to(torch.bfloat16), torch.zeros((8, 64), device="cuda")
    side = torch.cuda.Stream()
    spmm = lambda **k: tm.tmask_spmm24(*[{"vals": vals, "idx": idx, "rows": 64, "cols": 128, "x": x, "y": y, **k}[n]
                                         for n in ("vals", "idx", "rows", "cols", "x", "y")], stream=k.get("stream"))
    calls = [
        lambda: tm.tmask_approx(batch, None, 2, 4, workspace=wsp), lambda: tm.tmask_exact(batch, None, 4, 8, workspace=wsp, stream=side),
        lambda: tm.tmask_prune_1d(batch, None, 2, 4, workspace=wsp), lambda: tm.tmask_approx(batch, None, 3, 5, workspace=wsp),
        lambda: tm.tmask_approx(batch, None, 2, 4), lambda: tm.tmask_approx(batch, None, 2, 4, workspace=wsp[:64]),
        lambda: tm.tmask_approx(batch, None, 2, 4, workspace=7), lambda: tm.tmask_approx(batch, None, 2.0, 4, workspace=wsp),
        lambda: tm.tmask_approx(batch, None, 2, 4, workspace=wsp, stream=7), lambda: tm.tmask_approx(batch, None, 2, 4, mask_fmt=9, workspace=wsp),
        lambda: tm.tmask_approx_dense(w, None, dst, 2, 4), lambda: tm.tmask_approx_dense(w, None, dst, 4, 4),
        lambda: tm.tmask_score(batch, None, 2, 4, out, per_block_obj=per, workspace=wsp), lambda: tm.tmask_score(batch, None, 2, 4, out, workspace=wsp),
        lambda: tm.tmask_score(batch, None, 2, 4, out[:8], workspace=wsp), lambda: tm.tmask_score(batch, None, 2, 4, out.cpu(), workspace=wsp),
        lambda: tm.tmask_score(batch, None, 2, 4, out, per_block_obj=per.double(), workspace=wsp),
        lambda: spmm(), lambda: spmm(stream=side), lambda: spmm(x=x.float()), lambda: spmm(y=y.half()), lambda: spmm(idx=idx[:, :8]),
        lambda: spmm(vals=vals.t()), lambda: spmm(x=x[:, ::2]), lambda: spmm(y=y.cpu()), lambda: spmm(rows=60), lambda: spmm(cols=64),
        lambda: spmm(y=y[:, :32]), lambda: spmm(x=x[0]), lambda: spmm(x=torch.nn.Parameter(x)), lambda: spmm(y=torch.zeros((8, 66), device="cuda")[:, :64])]
    kept = [masks[0], obj, out, per, dst[0], y]
    seen = set()
    for k, call in enumerate(calls):
        got = []
        for half in (native, NONE):
            monkeypatch.setattr(tm, "_calls", half)
            for t in kept:
                t.zero_()
            masks[0].fill_(1)
            torch.cuda.synchronize()
            got.append((_outcome(call), [t.clone() for t in kept]))
        assert got[0][0] == got[1][0], k
        assert all(torch.equal(a, b) for a, b in zip(got[0][1], got[1][1])), k
        seen.add(None if got[0][0] is None else got[0][0][0])
    assert {None, tm.TmaskError, TypeError, ValueError} <= seen
    assert lib is tm.load_library()
