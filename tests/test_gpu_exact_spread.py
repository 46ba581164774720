"""tmask_exact at M = 8 and 16, and Algorithm 1 for bf16 at M = 16, have two kernels: calls that leave the chip idle give each column
of a block a lane, all others four (eight) columns; so do several matrices of tmask_exact that the first kernel would need a
second launch for.  Both against the oracle on the same matrices, alone and beside a large one; and the first where the workspace has
no room for its records: a second launch, or workgroups of 512 threads.  What a call changes in its workspace shows which way it went."""
import numpy as np
import pytest

import oracle
from paper_2102_08124_amd import workloads as wl

from .test_gpu_parity import _check_exact

pytestmark = pytest.mark.gpu

tm = pytest.importorskip("paper_2102_08124_amd.binding")
torch = pytest.importorskip("torch")
from .gpu_util import mask_to_host, run_masks, to_dev  # noqa: E402


def _kinds(M, dt):
    """One block; a workgroup of 256 columns less a block, full and one block more; several block-rows; and blocks that the start
    leaves unbalanced: tied values, zeros, rows and columns scaled, columns alike."""
    rng = np.random.default_rng(300 + M)
    f = lambda r, c, s: wl.gaussian_f32(r, c, seed=301 + M + s)
    sparse = f(3 * M, 21 * M, 5)
    sparse[rng.random(sparse.shape) < 0.6] = 0
    rows = f(2 * M, 33 * M, 6) * np.exp2(rng.integers(-20, 21, size=(2 * M, 1))).astype(np.float32)
    alike = np.repeat(np.abs(f(2 * M, 17, 7)), M, axis=1) + np.float32(0.001) * np.abs(f(2 * M, 17 * M, 8))
    ws = [f(M, M, 0), f(M, 256 - M, 1), f(M, 256, 2), f(M, 256 + M, 3), f(5 * M, 7 * M, 4),
          wl.tie_heavy_f32(3 * M, 21 * M, 302, levels=3), sparse, rows, alike]
    return [np.ascontiguousarray(w if dt == "f32" else wl.f32_to_bf16_bits(w)) for w in ws]


def _changed(call, wsp):
    """Runs a call with objectives on a workspace full of ones.  (True, words): it added up its sums itself, and cleared a record of two
    words of 64 bits for each workgroup but a matrix' last; (False, words): it left a result of one word for each workgroup."""
    wsp.fill_(0xFF)
    call()
    torch.cuda.synchronize()
    words = wsp[:wsp.numel() // 8 * 8].view(torch.int64)
    words = words[words != -1]
    return not bool(words.any()), words.numel()


def _run(find, ws, N, M, fmt, columns, threads=256):
    """Masks and objectives, and (in one launch, changed words) as they are for workgroups of so many lanes, each holding so many columns."""
    dev = [to_dev(w, ld=w.shape[1] + 16) for w in ws]
    masks, obj, wsp = tm.alloc_masks(dev, fmt), torch.full((len(ws),), -1.0, dtype=torch.float64, device="cuda"), tm.alloc_workspace(dev, N, M)
    for m in masks:
        m.fill_(0xCD)
    itself, words = _changed(lambda: find(dev, masks, N, M, objective=obj, mask_fmt=fmt, workspace=wsp), wsp)
    per = [-(-w.size // (M * columns * threads)) for w in ws]
    assert words == (sum(2 * (n - 1) for n in per) if itself else sum(per)), (itself, words, per)
    return [mask_to_host(m, w.shape[1], fmt) for m, w in zip(masks, ws)], obj.cpu().numpy(), itself


def _large(dt):
    """Beside it no small matrix gets a column per lane: its records would not fit (M = 16), or there are too many workgroups (M = 8)."""
    w = wl.gaussian_f32(1024, 1040, seed=311)
    return w if dt == "f32" else wl.f32_to_bf16_bits(w)


@pytest.mark.parametrize("fmt", [tm.TMASK_MASK_U8, tm.TMASK_MASK_BITS])
@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("N,M", [(4, 8), (1, 8), (6, 8), (8, 16), (3, 16), (15, 16)])
def test_both_kernels_against_the_oracle(N, M, dt, fmt):
    ws = _kinds(M, dt)
    together, sums = [], []
    for part in (ws[:5], ws[5:]):
        masks, obj, _ = _run(tm.tmask_exact, part + [_large(dt)], N, M, fmt, 4)
        together += masks[:-1]
        sums += list(obj[:-1])
    for k, w in enumerate(ws):
        (alone,), own, _ = _run(tm.tmask_exact, [w], N, M, fmt, 1)
        _, total, per_block = oracle.exact(w, N, M, per_block=True, threads=8)
        for mask, s in ((alone, own[0]), (together[k], sums[k])):
            _check_exact(w, mask, N, M, per_block)
            assert s == pytest.approx(total, rel=1e-5)


@pytest.mark.parametrize("fmt", [tm.TMASK_MASK_U8, tm.TMASK_MASK_BITS])
@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("N,M", [(4, 8), (1, 8), (7, 8), (8, 16), (1, 16), (15, 16)])
def test_more_unbalanced_blocks_than_search_slots_on_the_strips(N, M, dt, fmt):
    # 195 blocks (M = 8: 128 to a workgroup of strips, M = 16: 64; 32 and 16 are searched at a time), most of them left unbalanced
    rng = np.random.default_rng(1700 + N + M)
    rows, cols = 3 * M, 65 * M
    base = wl.gaussian_f32(rows, cols, seed=1701 + M)
    ws = [np.where(rng.random(base.shape) < 0.5, np.float32(0), base), wl.tie_heavy_f32(rows, cols, 1702, levels=3),
          base * np.exp2(rng.integers(-20, 21, size=(rows, 1))).astype(np.float32)]
    if dt == "bf16":
        ws = [wl.f32_to_bf16_bits(w) for w in ws]
    masks, obj, _ = _run(tm.tmask_exact, ws + [_large(dt)], N, M, fmt, 4)
    for w, mask, s in zip(ws, masks, obj):
        _, total, per_block = oracle.exact(w, N, M, per_block=True, threads=8)
        _check_exact(w, mask, N, M, per_block)
        assert s == pytest.approx(total, rel=1e-5)


@pytest.mark.parametrize("fmt", [tm.TMASK_MASK_U8, tm.TMASK_MASK_BITS])
@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("N,M", [(4, 8), (3, 8), (8, 16), (5, 16), (15, 16)])
def test_a_matrix_has_the_same_mask_in_every_call(N, M, dt, fmt):
    """Where masks are equally good, too, the choice depends neither on the other matrices of the call nor on the objectives: alone with
    and without one (a column to a lane), and beside a matrix with which the call takes four columns to a lane."""
    rng = np.random.default_rng(320 + M)
    f = lambda s: wl.gaussian_f32(12 * M, 33 * M, seed=321 + M + s)
    sparse = f(0)
    sparse[rng.random(sparse.shape) < 0.6] = 0
    mixed = np.where((np.arange(33 * M) // M % 3 == 0)[None, :], wl.tie_heavy_f32(12 * M, 33 * M, 322, levels=2), f(1))
    ws = [sparse, mixed, f(2), wl.tie_heavy_f32(12 * M, 33 * M, 323, levels=3)]
    ws = _kinds(M, dt) + [w if dt == "f32" else wl.f32_to_bf16_bits(w) for w in ws]
    for k, w in enumerate(ws):
        (alone,), _, _ = _run(tm.tmask_exact, [w], N, M, fmt, 1)
        (bare,), _ = run_masks(tm.tmask_exact, [w], N, M, fmt, with_objective=False)
        (beside, _), _, _ = _run(tm.tmask_exact, [w, _large(dt)], N, M, fmt, 4)
        assert np.array_equal(alone, bare), k
        assert np.array_equal(alone, beside), k


def _check(w, mask, total, N, M, exact):
    want, best, *per_block = oracle.exact(w, N, M, per_block=True, threads=8) if exact else oracle.approx(w, N, M)
    if exact:
        _check_exact(w, mask, N, M, per_block[0])
    else:
        assert np.array_equal(mask, want)
    if np.isfinite(best):
        assert total == pytest.approx(best, rel=1e-5)


# The workspace has 56 bytes for 1024 columns of a block-row, and 256, where a column per lane leaves records of 64.
@pytest.mark.parametrize("fmt", [tm.TMASK_MASK_U8, tm.TMASK_MASK_BITS])
@pytest.mark.parametrize("find,dt,N,M,rows,cols,threads,itself", [
    ("exact", "f32", 8, 16, 512, 1024, 256, True), ("exact", "bf16", 5, 16, 512, 1024, 256, True),
    ("exact", "f32", 8, 16, 512, 1056, 256, False), ("exact", "bf16", 5, 16, 512, 1056, 256, False),
    ("exact", "f32", 4, 8, 512, 512, 256, True), ("exact", "bf16", 3, 8, 512, 512, 256, True),
    ("exact", "f32", 4, 8, 512, 528, 512, True), ("exact", "f32", 3, 8, 512, 528, 512, True), ("exact", "bf16", 4, 8, 512, 528, 512, True),
    ("exact", "bf16", 3, 8, 1024, 512, 512, True), ("exact", "f32", 4, 8, 1024, 1016, 512, True),
    ("approx", "bf16", 8, 16, 512, 1024, 256, True), ("approx", "bf16", 8, 16, 512, 1056, 512, True),
    ("approx", "bf16", 5, 16, 512, 1056, 512, True), ("approx", "bf16", 8, 16, 1024, 1024, 512, True)])
def test_with_and_without_room_for_the_records(find, dt, N, M, rows, cols, threads, itself, fmt):
    w = wl.gaussian_f32(rows, cols, seed=310)
    w[:M] = wl.tie_heavy_f32(M, cols, 310, levels=3)
    w = w if dt == "f32" else wl.f32_to_bf16_bits(w)
    (mask,), obj, one = _run(tm.tmask_exact if find == "exact" else tm.tmask_approx, [w], N, M, fmt, 1, threads)
    assert one == itself
    _check(w, mask, obj[0], N, M, find == "exact")


@pytest.mark.parametrize("fmt", [tm.TMASK_MASK_U8, tm.TMASK_MASK_BITS])
@pytest.mark.parametrize("N", [8, 13])
def test_workgroups_of_512_threads_over_several_matrices(N, fmt):
    ws = [wl.f32_to_bf16_bits(w) for w in (wl.gaussian_f32(512, 1056, seed=330), wl.gaussian_f32(16, 16, seed=331), wl.tie_heavy_f32(48, 336, 332, levels=3),
                                           wl.gaussian_f32(16, 528, seed=333), wl.gaussian_f32(272, 1024, seed=334))]
    masks, obj, itself = _run(tm.tmask_approx, ws, N, 16, fmt, 1, 512)
    assert itself
    for w, mask, total in zip(ws, masks, obj):
        _check(w, mask, total, N, 16, False)


@pytest.mark.parametrize("fmt", [tm.TMASK_MASK_U8, tm.TMASK_MASK_BITS])
@pytest.mark.parametrize("N", [8, 5, 15])
def test_algorithm_1_for_bf16_at_m16_on_the_strips(N, fmt):
    """4096 x 2064: one workgroup of columns more than eight to each of 256 compute units."""
    odd = wl.gaussian_f32(32, 272, seed=313)
    odd[::5, ::3], odd[1::7], odd[:, 5] = np.inf, np.nan, -0.0
    ws = [wl.f32_to_bf16_bits(w) for w in (wl.tie_heavy_f32(48, 336, 312, levels=3), odd, wl.gaussian_f32(4096, 2064, seed=335))]
    masks, obj, _ = _run(tm.tmask_approx, ws, N, 16, fmt, 8)
    dev = [to_dev(w) for w in ws]
    outs, copies = [torch.full(w.shape, 7.0, dtype=torch.bfloat16, device="cuda") for w in ws], tm.alloc_masks(dev, fmt)
    tm.tmask_approx_dense(dev, copies, outs, N, 16, mask_fmt=fmt)
    torch.cuda.synchronize()
    for w, mask, total, out, copy in zip(ws, masks, obj, outs, copies):
        _check(w, mask, total, N, 16, False)
        assert np.array_equal(mask_to_host(copy, w.shape[1], fmt), mask)
        assert np.array_equal(out.view(torch.int16).cpu().numpy(), np.where(mask != 0, w, np.uint16(0)).view(np.int16))


@pytest.mark.parametrize("fmt", [tm.TMASK_MASK_U8, tm.TMASK_MASK_BITS])
@pytest.mark.parametrize("N", [8, 1, 6, 15])
def test_algorithm_1_for_bf16_at_m16(N, fmt):
    """A column per lane, with matrices of one block to 512 x 1040, and for ten of them in a call."""
    ties = wl.f32_to_bf16_bits(wl.tie_heavy_f32(48, 336, 312, levels=3))
    odd = wl.gaussian_f32(32, 272, seed=313)
    odd[::5, ::3], odd[1::7], odd[:, 5] = np.inf, np.nan, -0.0
    odd = wl.f32_to_bf16_bits(odd)
    plain = [wl.f32_to_bf16_bits(wl.gaussian_f32(r, c, seed=314 + c)) for r, c in ((16, 16), (16, 256), (16, 272), (512, 1024), (512, 1040))]
    for ws in [[w] for w in plain] + [[ties], [odd], plain[:2] + [ties, odd], plain[:3] * 3 + [ties]]:
        masks, obj = run_masks(tm.tmask_approx, ws, N, 16, fmt, ld_pad=16)
        for k, w in enumerate(ws):
            want, total = oracle.approx(w, N, 16)
            assert np.array_equal(masks[k], want), k
            if np.isfinite(total):
                assert obj[k] == pytest.approx(total, rel=1e-5)
            dev = to_dev(w, ld=w.shape[1] + 8)
            out, mask = torch.full(w.shape, 7.0, dtype=torch.bfloat16, device="cuda"), tm.alloc_masks([dev], fmt)
            tm.tmask_approx_dense([dev], mask, [out], N, 16, mask_fmt=fmt)
            alone = out.clone().fill_(3.0)
            tm.tmask_approx_dense([dev], None, [alone], N, 16, mask_fmt=fmt)
            torch.cuda.synchronize()
            assert np.array_equal(mask_to_host(mask[0], w.shape[1], fmt), want)
            bits = np.where(want != 0, w, np.uint16(0)).view(np.int16)
            for o in (out, alone):
                assert np.array_equal(o.view(torch.int16).cpu().numpy(), bits)
