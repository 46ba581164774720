"""Where the compressed outputs' lines start at odd bytes and end in the middle of a tile: every byte against the oracle, and none
outside the outputs."""
import numpy as np
import pytest

import oracle
from paper_2102_08124_amd import workloads as wl

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
tm = pytest.importorskip("paper_2102_08124_amd.binding")
from .gpu_util import mask_to_dev, to_dev  # noqa: E402

GUARD = 64


def _guarded(shapes, kinds):
    """Outputs with guard bytes around each, in one buffer of 0xEE."""
    sizes = [int(np.prod(s)) * torch.empty(0, dtype=k).element_size() for s, k in zip(shapes, kinds)]
    steps = [GUARD + -(-n // GUARD) * GUARD for n in sizes]
    flat = torch.full((sum(steps) + GUARD,), 0xEE, dtype=torch.uint8, device="cuda")
    views, used, at = [], np.zeros(flat.numel(), bool), GUARD
    for shape, kind, n, step in zip(shapes, kinds, sizes, steps):
        views.append(flat[at:at + n].view(kind).view(shape))
        used[at:at + n] = True
        at += step
    return flat, tuple(views), used


def _check(flat, views, used, want):
    host = flat.cpu().numpy()
    for view, w, name in zip(views, want, ("vals", "idx", "valsT", "idxT")):
        got = view.contiguous().view(-1).view(torch.uint8).cpu().numpy()
        assert np.array_equal(got, np.ascontiguousarray(w).view(np.uint8).ravel()), name
    assert (host[~used] == 0xEE).all()


@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("N,M", [(2, 4), (1, 4), (4, 8), (2, 8), (3, 8), (7, 8), (8, 16), (3, 16), (15, 16), (16, 32)])
@pytest.mark.parametrize("rows,cols", [(1, 1), (1, 3), (3, 1), (5, 33), (17, 9), (9, 41)])          # in blocks
@pytest.mark.parametrize("copies", [1, 9])                       # workgroups of 1024 threads, of 256
def test_lines_at_odd_bytes(N, M, dt, rows, cols, copies):
    if dt == "bf16" and M == 4:
        cols = 2 * cols                                          # the tiled kernels: rows of whole 16 bytes
    w = wl.gaussian_f32(rows * M, cols * M, seed=50 + rows)
    w = w if dt == "f32" else wl.f32_to_bf16_bits(w)
    mask, total = oracle.approx(w, N, M)
    want = oracle.apply_pack(w, mask, N, M)
    dev, dmask = to_dev(w), mask_to_dev(mask, tm.TMASK_MASK_U8)
    kinds = [dev.dtype, torch.uint8, dev.dtype, torch.uint8]
    flat, views, used = _guarded(tm.packed_shapes(*w.shape, N, M), kinds)
    others = [tm.alloc_packed(dev, N, M) for _ in range(copies - 1)]
    tm.tmask_apply_pack([dev] * copies, [dmask] * copies, [views] + others, N, M)
    torch.cuda.synchronize()
    _check(flat, views, used, want)
    if copies > 1:
        return
    flat, views, used = _guarded(tm.packed_shapes(*w.shape, N, M), kinds)
    obj, wsp = torch.zeros(1, dtype=torch.float64, device="cuda"), tm.alloc_workspace([dev], N, M)
    tm.tmask_approx_pack([dev], tm.alloc_masks([dev]), [views], N, M, objective=obj, workspace=wsp)
    torch.cuda.synchronize()
    _check(flat, views, used, want)
    assert float(obj[0]) == pytest.approx(total, rel=1e-5)


@pytest.mark.parametrize("dt,N,M", [("f32", 4, 8), ("f32", 2, 4), ("bf16", 2, 4), ("bf16", 4, 8)])
@pytest.mark.parametrize("copies", [3, 8, 9, 15, 17, 23, 25, 31, 33, 39, 41, 79, 81])   # 16 (bf16: 8) tiles each: either side of the lines
def test_quarter_half_and_whole_tiles(dt, N, M, copies):                                # between quarter, half and whole tiles
    w = wl.gaussian_f32(200, 776, seed=57)
    w = w if dt == "f32" else wl.f32_to_bf16_bits(w)
    mask, total = oracle.approx(w, N, M)
    want = [torch.from_numpy(np.ascontiguousarray(o).view(np.uint8)).cuda() for o in oracle.apply_pack(w, mask, N, M)]
    ws, masks = [to_dev(w)] * copies, [mask_to_dev(mask, tm.TMASK_MASK_U8)] * copies
    packed, fused = ([tm.alloc_packed(x, N, M) for x in ws] for _ in range(2))
    obj, wsp = torch.zeros(copies, dtype=torch.float64, device="cuda"), tm.alloc_workspace(ws, N, M)
    tm.tmask_apply_pack(ws, masks, packed, N, M)
    tm.tmask_approx_pack(ws, None, fused, N, M, objective=obj, workspace=wsp)
    torch.cuda.synchronize()
    for p in packed + fused:
        for got, o in zip(p, want):
            assert torch.equal(got.view(torch.uint8), o)
    assert obj.cpu().numpy() == pytest.approx(np.full(copies, total), rel=1e-5)


@pytest.mark.parametrize("rows,cols", [(1000, 1028), (2048, 2052)])                     # quarter and half tiles of narrow strips
def test_narrow_strips_of_one_matrix(rows, cols):
    w = wl.f32_to_bf16_bits(wl.gaussian_f32(rows, cols, seed=58))
    mask, _ = oracle.approx(w, 2, 4)
    dev = to_dev(w)
    packed = tm.alloc_packed(dev, 2, 4)
    tm.tmask_apply_pack([dev], [mask_to_dev(mask, tm.TMASK_MASK_U8)], [packed], 2, 4)
    torch.cuda.synchronize()
    for got, o in zip(packed, oracle.apply_pack(w, mask, 2, 4)):
        assert torch.equal(got.view(torch.uint8), torch.from_numpy(np.ascontiguousarray(o).view(np.uint8)).cuda())
