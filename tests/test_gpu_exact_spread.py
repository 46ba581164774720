"""tmask_exact at M = 8 and 16 has two kernels: calls that leave the chip idle give each column of a block a lane, all others four
columns; so do several matrices that the first kernel would need a second launch for.  Both against the oracle on the same
matrices, alone and beside a large one, and what the first leaves to a second launch when the workspace has no room for its
records."""
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


@pytest.mark.parametrize("fmt", [tm.TMASK_MASK_U8, tm.TMASK_MASK_BITS])
@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("N,M", [(4, 8), (1, 8), (6, 8), (8, 16), (3, 16), (15, 16)])
def test_both_kernels_against_the_oracle(N, M, dt, fmt):
    ws = _kinds(M, dt)
    large = wl.gaussian_f32(512, 1040, seed=311)                 # with it the records of a column per lane do not fit
    large = large if dt == "f32" else wl.f32_to_bf16_bits(large)
    together, sums = [], []
    for part in (ws[:5], ws[5:]):
        masks, obj = run_masks(tm.tmask_exact, part + [large], N, M, fmt, ld_pad=16)
        together += masks[:-1]
        sums += list(obj[:-1])
    for k, w in enumerate(ws):
        (alone,), own = run_masks(tm.tmask_exact, [w], N, M, fmt, ld_pad=16)
        _, total, per_block = oracle.exact(w, N, M, per_block=True, threads=8)
        for mask, s in ((alone, own[0]), (together[k], sums[k])):
            _check_exact(w, mask, N, M, per_block)
            assert s == pytest.approx(total, rel=1e-5)


def _left(call, wsp):
    """How a call with objectives of one matrix went, by what it changes in a workspace full of ones: ("one launch", workgroups) if
    records of two words were there and are cleared, ("two", workgroups) if a result of each workgroup is left."""
    wsp.fill_(0xFF)
    call()
    torch.cuda.synchronize()
    words = wsp[:wsp.numel() // 8 * 8].view(torch.int64)
    changed = words[words != -1]
    if bool((changed == 0).all()):
        return "one launch", changed.numel() // 2 + 1
    return "two", changed.numel()


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
    large = wl.gaussian_f32(1024, 1040, seed=324)
    large = to_dev(large if dt == "f32" else wl.f32_to_bf16_bits(large))
    for k, w in enumerate(ws):
        (alone,), _ = run_masks(tm.tmask_exact, [w], N, M, fmt)
        (bare,), _ = run_masks(tm.tmask_exact, [w], N, M, fmt, with_objective=False)
        both = [to_dev(w), large]
        masks, obj, wsp = tm.alloc_masks(both, fmt), torch.zeros(2, dtype=torch.float64, device="cuda"), tm.alloc_workspace(both, N, M)
        _, workgroups = _left(lambda: tm.tmask_exact(both, masks, N, M, objective=obj, mask_fmt=fmt, workspace=wsp), wsp)
        # two matrices: one that waits in each that has two workgroups or more, and is counted once
        assert workgroups <= -(-w.size // (1024 * M)) + -(-1024 * 1040 // (1024 * M)) + 1
        assert np.array_equal(alone, bare), k
        assert np.array_equal(alone, mask_to_host(masks[0], w.shape[1], fmt)), k


@pytest.mark.parametrize("N,M,rows,cols", [(8, 16, 512, 1024), (8, 16, 512, 1040), (4, 8, 512, 512), (4, 8, 512, 520)])
@pytest.mark.parametrize("dt", ["f32", "bf16"])
def test_objective_with_and_without_room_for_the_records(N, M, rows, cols, dt):
    # 32 workgroups of 256 strips of four columns have room for 128 records of 16 bytes, one more has not: a second launch at M =
    # 16, workgroups of 512 threads at M = 8
    w = wl.gaussian_f32(rows, cols, seed=310)
    w = w if dt == "f32" else wl.f32_to_bf16_bits(w)
    (mask,), obj = run_masks(tm.tmask_exact, [w], N, M)
    mag = np.abs(w if dt == "f32" else (w.astype(np.uint32) << 16).view(np.float32)).astype(np.float64)
    # masks are checked above; a wavefront's 64 columns are added in fp32, at most M + 6 additions deep
    assert obj[0] == pytest.approx((mag * mask).sum(), rel=(M + 6) * 2.0 ** -24)


@pytest.mark.parametrize("fmt", [tm.TMASK_MASK_U8, tm.TMASK_MASK_BITS])
@pytest.mark.parametrize("N", [8, 1, 6, 15])
def test_algorithm_1_for_bf16_at_m16(N, fmt):
    """A column per lane up to 512 x 1024 (workgroups of 256 threads), 512 x 1040 (512) and for nine matrices; larger ones on the strips."""
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
