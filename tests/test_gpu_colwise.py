"""GPU parity for the column-per-lane kernels: M = 32 on every entry point, and M = 4, 8, 16 on matrices that only
satisfy the paper's own requirement (rows and cols multiples of M; Sec. 4) but miss the 16-byte alignment of the strip
kernels: odd leading dimensions, views that start at an odd element, bf16 widths with cols % 8 == 4, masks and packed
outputs at odd byte offsets.  Same bars as everywhere: approximation / row pruning bit-exact, exact masks valid with
every block's retained L1 within 1e-5 of the oracle's, scores exact in the counts, packed operands byte-exact."""
import numpy as np
import pytest

import oracle
from paper_2102_08124_amd import workloads as wl
from tests import refs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2102_08124_amd import binding as tm                                   # noqa: E402
from tests.gpu_util import run_masks, run_score, run_pack, run_fused, to_dev, mask_to_host   # noqa: E402

FMTS = [tm.TMASK_MASK_U8, tm.TMASK_MASK_BITS]


def _inputs(kind, rows, cols, seed):
    if kind == "f32":
        return wl.gaussian_f32(rows, cols, seed)
    if kind == "bf16":
        return wl.f32_to_bf16_bits(wl.gaussian_f32(rows, cols, seed, std=0.02))
    if kind == "ties":
        return wl.tie_heavy_f32(rows, cols, seed, levels=4)
    if kind == "ties_bf16":
        return wl.f32_to_bf16_bits(wl.tie_heavy_f32(rows, cols, seed, levels=3))
    if kind == "special":
        return wl.special_values_f32(rows, cols, seed)
    raise ValueError(kind)


def _check_exact(w, mask, N, M, oracle_pb):
    b = refs.to_blocks(mask, M)
    assert np.all(b.sum(axis=3) == N) and np.all(b.sum(axis=2) == N), "mask is not exactly N per row/column"
    got = refs.per_block_sums(refs.magnitudes(w) * mask, M)
    np.testing.assert_allclose(got, oracle_pb, rtol=1e-5, atol=1e-30)


# ---------------------------------------------------------------- M = 32 ------------------------

@pytest.mark.parametrize("fmt", FMTS)
@pytest.mark.parametrize("N", [16, 5, 27])
@pytest.mark.parametrize("kind", ["f32", "bf16", "ties", "ties_bf16", "special"])
def test_m32_approx_and_row_pruning_bit_exact(kind, N, fmt):
    # 3 block-rows x 416 columns: 6.5 tiles of 64 columns per block-row (a half-filled last tile), several workgroups
    w = _inputs(kind, 96, 416, seed=3200 + N)
    (mask,), obj = run_masks(tm.tmask_approx, [w], N, 32, fmt)
    omask, oobj = oracle.approx(w, N, 32)
    assert np.array_equal(mask, omask)
    if kind != "special":
        assert obj[0] == pytest.approx(oobj, rel=1e-5)
    (mask,), obj = run_masks(tm.tmask_prune_1d, [w], N, 32, fmt)
    omask, oobj = oracle.prune_1d(w, N, 32)
    assert np.array_equal(mask, omask)
    if kind != "special":
        assert obj[0] == pytest.approx(oobj, rel=1e-5)


@pytest.mark.parametrize("dt", ["f32", "bf16"])
def test_m32_batch_of_matrices_with_strides(dt):
    shapes = [(32, 32), (64, 32), (32, 96), (128, 160), (32, 1056)]
    ws = [_inputs(dt, *shapes[k % len(shapes)], seed=3300 + k) for k in range(9)]
    masks, obj = run_masks(tm.tmask_approx, ws, 16, 32, ld_pad=24)
    for k, w in enumerate(ws):
        omask, oobj = oracle.approx(w, 16, 32)
        assert np.array_equal(masks[k], omask), "matrix %d" % k
        assert obj[k] == pytest.approx(oobj, rel=1e-5)


@pytest.mark.parametrize("fmt", FMTS)
@pytest.mark.parametrize("N", [16, 9, 30])
@pytest.mark.parametrize("kind", ["f32", "bf16", "ties"])
def test_m32_exact_optimal(kind, N, fmt):
    w = _inputs(kind, 64, 160, seed=3400 + N)             # 2 x 5 blocks, the last tile half filled
    (mask,), obj = run_masks(tm.tmask_exact, [w], N, 32, fmt)
    _, oobj, opb = oracle.exact(w, N, 32, per_block=True)
    _check_exact(w, mask, N, 32, opb)
    assert obj[0] == pytest.approx(oobj, rel=1e-5)


def test_m32_exact_structured_blocks():
    # blocks that need long augmenting chains: heavy entries concentrated in a few rows, all-equal and all-zero blocks
    rng = np.random.default_rng(3500)
    w = rng.standard_normal((64, 128)).astype(np.float32)
    w[:8, :32] *= 100.0                   # eight heavy rows: every column wants to keep the same rows
    w[:, 40:44] *= 50.0                   # heavy columns
    w[32:, 64:96] = 1.0                   # all equal
    w[32:, 96:] = 0.0                     # all zero
    for N in (16, 4):
        (mask,), obj = run_masks(tm.tmask_exact, [w], N, 32)
        _, oobj, opb = oracle.exact(w, N, 32, per_block=True)
        _check_exact(w, mask, N, 32, opb)
        assert obj[0] == pytest.approx(oobj, rel=1e-5)


@pytest.mark.parametrize("fmt", FMTS)
@pytest.mark.parametrize("dt", ["f32", "bf16"])
def test_m32_score_and_pack_match_oracle(dt, fmt):
    N, M = 16, 32
    w = _inputs(dt, 96, 288, seed=3600)
    amask, _ = oracle.approx(w, N, M)             # keeps fewer than N in places: fillers
    emask, _ = oracle.exact(w, N, M)
    bad = emask.copy()
    bad[0, :40] = 1                               # rows / columns with more than N kept
    for mask in (amask, emask, bad):
        (sc,), (pb,) = run_score([w], [mask], N, M, fmt)
        o = oracle.score(w, mask, N, M)
        assert (sc["kept"], sc["row_violations"], sc["col_violations"], sc["row_not_n"], sc["col_not_n"]) == \
               (o.kept, o.row_violations, o.col_violations, o.row_not_n, o.col_not_n)
        assert sc["retained_l1"] == pytest.approx(o.retained_l1, rel=1e-5)
        assert sc["total_l1"] == pytest.approx(o.total_l1, rel=1e-5)
        np.testing.assert_allclose(pb, o.per_block, rtol=1e-5, atol=1e-30)
    for mask, NN in ((amask, N), (emask, N), (oracle.approx(w, 5, M)[0], 5)):
        (got,) = run_pack([w], [mask], NN, M, fmt)
        want = oracle.apply_pack(w, mask, NN, M)
        for g, t in zip(got, want):
            assert np.array_equal(g.view(np.uint8), t.view(np.uint8))


@pytest.mark.parametrize("fmt", FMTS)
@pytest.mark.parametrize("dt", ["f32", "bf16"])
def test_m32_tiled_pack_ragged_tiles_and_degenerate_masks(dt, fmt):
    """16:32 on matrices aligned for 16-byte loads runs the tiled pack kernel (64 rows x 256 bytes per tile): tiles cut
    by the matrix edge in both directions, padded rows, and masks that keep too many, too few, all or nothing."""
    N, M = 16, 32
    rng = np.random.default_rng(3650)
    ws, masks = [], []
    for k, (rows, cols) in enumerate([(32, 32), (64, 64), (96, 160), (160, 416), (32, 1056)]):
        w = _inputs(dt, rows, cols, seed=3651 + k)
        ws += [w, w, w]
        masks += [(rng.random(w.shape) < 0.5).astype(np.uint8), np.zeros(w.shape, np.uint8), np.ones(w.shape, np.uint8)]
    for pad in (0, 24):
        got = run_pack(ws, masks, N, M, fmt, ld_pad=pad)
        for k, (w, m) in enumerate(zip(ws, masks)):
            want = oracle.apply_pack(w, m, N, M)
            for g, t in zip(got[k], want):
                assert np.array_equal(g.view(np.uint8), t.view(np.uint8)), (k, pad)


def test_m32_approx_pack_and_dense_calls():
    N, M = 16, 32
    for dt in ("f32", "bf16"):
        w = _inputs(dt, 64, 224, seed=3700)
        omask, oobj = oracle.approx(w, N, M)
        (got,), (mask,), obj = run_fused([w], N, M)
        assert np.array_equal(mask, omask) and obj[0] == pytest.approx(oobj, rel=1e-5)
        for g, t in zip(got, oracle.apply_pack(w, omask, N, M)):
            assert np.array_equal(g.view(np.uint8), t.view(np.uint8))
        wd = to_dev(w)
        out = torch.empty_like(wd)
        m = tm.alloc_masks([wd])[0]
        tm.tmask_approx_dense([wd], [m], [out], N, M)
        torch.cuda.synchronize()
        raw = wd.view(torch.int16 if dt == "bf16" else torch.int32).cpu().numpy()
        got_out = out.view(torch.int16 if dt == "bf16" else torch.int32).cpu().numpy()
        assert np.array_equal(m.cpu().numpy(), omask)
        assert np.array_equal(got_out, np.where(omask != 0, raw, 0))
        # row pruning with the mean of the pruned weights absorbed (Sec. 5), no mask written
        tm.tmask_prune_1d_dense([wd], None, [out], N, M, absorb_mean=True)
        torch.cuda.synchronize()
        pmask, _ = oracle.prune_1d(w, N, M)
        wf = wl.bf16_bits_to_f32(w) if dt == "bf16" else w
        want = oracle.apply_dense(wf, pmask, M, absorb_mean=True)
        got_f = out.float().cpu().numpy().astype(np.float64)
        tol = 2.0 ** -20 * np.abs(wf.astype(np.float64)).reshape(64, -1, M).sum(2).repeat(M, axis=1)
        if dt == "bf16":
            tol = tol + 2.0 ** -8 * np.abs(want)
        assert np.all(np.abs(got_f - want) <= tol + 1e-30)


@pytest.mark.parametrize("fmt", FMTS)
@pytest.mark.parametrize("kind", ["bf16", "ties_bf16", "zeros", "special"])
def test_m32_bf16_by_rows_and_by_columns(kind, fmt):
    """16:32 of aligned bf16 matrices is read by rows, two keys to a register; one pitch that is odd sends the whole batch
    the column-per-lane way.  Both against the oracle: half tiles, one block, more block-rows than one XCD takes."""
    hs = []
    for k, (rows, cols) in enumerate([(32, 32), (32, 96), (96, 416), (320, 1056)]):
        w = _inputs({"zeros": "bf16", "special": "special"}.get(kind, kind), rows, cols, seed=3230 + k)
        w = w if w.dtype == np.uint16 else wl.f32_to_bf16_bits(w)
        hs.append(np.where(wl.f32_to_bf16_bits(wl.gaussian_f32(rows, cols, 3240 + k)) & 0x4000, w, 0x8000) if kind == "zeros" else w)
    hs = [h.astype(np.uint16) for h in hs]
    want = [oracle.approx(h, 16, 32) for h in hs]
    for pad in (0, 8, 1):
        got, obj = run_masks(tm.tmask_approx, hs, 16, 32, fmt, ld_pad=pad)
        for g, o, (om, oo) in zip(got, obj, want):
            assert np.array_equal(g, om)
            if kind != "special":
                assert o == pytest.approx(oo, rel=1e-5)
        got, _ = run_masks(tm.tmask_approx, hs, 16, 32, fmt, ld_pad=pad, with_objective=False)
        for g, (om, _) in zip(got, want):
            assert np.array_equal(g, om)


def test_m32_argument_errors():
    w = torch.zeros((64, 64), dtype=torch.float32, device="cuda")
    m = tm.alloc_masks([w])[0]
    with pytest.raises(tm.TmaskError) as e:
        tm.tmask_approx([w], [m], 32, 32)
    assert e.value.code == tm.TMASK_ERR_NM
    with pytest.raises(tm.TmaskError) as e:
        tm.tmask_approx([w[:48]], [m[:48]], 16, 32)          # 48 rows: not a multiple of 32
    assert e.value.code == tm.TMASK_ERR_SHAPE
    torch.cuda.synchronize()


# ---------------------------------------------------------------- unaligned, M = 4, 8, 16 --------

def _unaligned_dev(w_np, ld, off):
    """Device view of w_np inside a wider buffer: row stride ld elements, first element `off` elements in."""
    rows, cols = w_np.shape
    if w_np.dtype == np.uint16:
        t = torch.from_numpy(w_np.view(np.int16)).view(torch.bfloat16)
    else:
        t = torch.from_numpy(w_np)
    flat = torch.zeros(rows * ld + off, dtype=t.dtype, device="cuda")
    view = flat[off:].view(rows, ld)[:, :cols]
    view.copy_(t.cuda())
    return view


def _unaligned_masks(ws, fmt, mld_extra, moff):
    out = []
    for w in ws:
        r, c = tm.mask_shape(w.shape[0], w.shape[1], fmt)
        buf = torch.full((r, c + mld_extra + moff), 0xCD, dtype=torch.uint8, device="cuda")
        out.append(buf[:, moff:moff + c])
    return out


CASES_UNALIGNED = [
    # dtype, N, M, rows, cols, ld, element offset of the view
    ("bf16", 2, 4, 16, 36, 36, 0),        # bf16 cols % 8 == 4: 72-byte rows
    ("bf16", 2, 4, 24, 260, 263, 1),      # odd leading dimension and an odd first element
    ("f32", 2, 4, 20, 132, 133, 0),       # fp32 with an odd leading dimension
    ("f32", 2, 4, 16, 64, 64, 1),         # aligned pitch, view starts 4 bytes in
    ("bf16", 4, 8, 24, 264, 270, 3),
    ("f32", 4, 8, 16, 136, 139, 2),
    ("f32", 3, 8, 16, 72, 73, 0),
    ("bf16", 8, 16, 32, 272, 277, 5),
    ("f32", 8, 16, 32, 144, 147, 1),
    ("ties", 2, 4, 16, 68, 71, 1),
]


@pytest.mark.parametrize("fmt", FMTS)
@pytest.mark.parametrize("kind,N,M,rows,cols,ld,off", CASES_UNALIGNED)
def test_unaligned_masks_scores_and_packs(kind, N, M, rows, cols, ld, off, fmt):
    if fmt == tm.TMASK_MASK_BITS and cols % 8:
        pytest.skip("bit masks need cols to be a multiple of 8")
    w = _inputs(kind, rows, cols, seed=3800 + cols)
    wd = _unaligned_dev(w, ld, off)
    assert wd.data_ptr() % 16 != 0 or (ld * wd.element_size()) % 16 != 0 or (cols * wd.element_size()) % 16 != 0
    obj = torch.full((3,), -1.0, dtype=torch.float64, device="cuda")
    wsp = tm.alloc_workspace([wd], N, M)
    masks = _unaligned_masks([wd] * 3, fmt, mld_extra=3, moff=1)
    tm.tmask_approx([wd], [masks[0]], N, M, objective=obj[0:1], mask_fmt=fmt, workspace=wsp)
    tm.tmask_exact([wd], [masks[1]], N, M, objective=obj[1:2], mask_fmt=fmt, workspace=wsp)
    tm.tmask_prune_1d([wd], [masks[2]], N, M, objective=obj[2:3], mask_fmt=fmt, workspace=wsp)
    torch.cuda.synchronize()
    got = [mask_to_host(m.contiguous(), cols, fmt) for m in masks]
    o = obj.cpu().numpy()
    amask, aobj = oracle.approx(w, N, M)
    assert np.array_equal(got[0], amask) and o[0] == pytest.approx(aobj, rel=1e-5)
    _, eobj, epb = oracle.exact(w, N, M, per_block=True)
    _check_exact(w, got[1], N, M, epb)
    assert o[1] == pytest.approx(eobj, rel=1e-5)
    pmask, pobj = oracle.prune_1d(w, N, M)
    assert np.array_equal(got[2], pmask) and o[2] == pytest.approx(pobj, rel=1e-5)
    # score of the approximate mask, read from its unaligned buffer
    sout = torch.zeros(tm.SCORE_OUT_BYTES, dtype=torch.uint8, device="cuda")
    pb = torch.full(((rows // M) * (cols // M),), -1.0, dtype=torch.float32, device="cuda")
    tm.tmask_score([wd], [masks[0]], N, M, sout, per_block_obj=pb, mask_fmt=fmt, workspace=wsp)
    torch.cuda.synchronize()
    sc = tm.read_scores(sout, 1)[0]
    so = oracle.score(w, amask, N, M)
    assert (sc["kept"], sc["row_violations"], sc["col_violations"], sc["row_not_n"], sc["col_not_n"]) == \
           (so.kept, so.row_violations, so.col_violations, so.row_not_n, so.col_not_n)
    assert sc["retained_l1"] == pytest.approx(so.retained_l1, rel=1e-5)
    np.testing.assert_allclose(pb.cpu().numpy().reshape(so.per_block.shape), so.per_block, rtol=1e-5, atol=1e-30)
    # apply + pack with the exact mask, and the two-step approx + pack
    for which, mask_dev, mask_np in (("apply_pack", masks[1], got[1]), ("approx_pack", masks[0], amask)):
        packed = tm.alloc_packed(wd, N, M)
        for t in packed:
            t.view(torch.uint8).fill_(0xEE)
        if which == "apply_pack":
            tm.tmask_apply_pack([wd], [mask_dev], [packed], N, M, mask_fmt=fmt)
        else:
            mask_dev.fill_(0xCD)
            tm.tmask_approx_pack([wd], [mask_dev], [packed], N, M, mask_fmt=fmt)
        torch.cuda.synchronize()
        want = oracle.apply_pack(w, mask_np, N, M)
        for g, t in zip(packed, want):
            gh = g.view(torch.int16).cpu().numpy().view(np.uint16) if g.dtype == torch.bfloat16 else g.cpu().numpy()
            assert np.array_equal(gh.view(np.uint8), t.view(np.uint8)), which


@pytest.mark.parametrize("kind,N,M,rows,cols,ld,off", CASES_UNALIGNED[:6])
def test_unaligned_dense_one_pass_calls(kind, N, M, rows, cols, ld, off):
    w = _inputs(kind, rows, cols, seed=3900 + cols)
    wd = _unaligned_dev(w, ld, off)
    outbuf = torch.zeros((rows, ld + 2), dtype=wd.dtype, device="cuda")
    out = outbuf[:, 1:1 + cols]
    tm.tmask_approx_dense([wd], None, [out], N, M)
    torch.cuda.synchronize()
    it = torch.int16 if wd.dtype == torch.bfloat16 else torch.int32
    raw = wd.contiguous().view(it).cpu().numpy()
    amask, _ = oracle.approx(w, N, M)
    assert np.array_equal(out.contiguous().view(it).cpu().numpy(), np.where(amask != 0, raw, 0))
    tm.tmask_prune_1d_dense([wd], None, [out], N, M, absorb_mean=False)
    torch.cuda.synchronize()
    pmask, _ = oracle.prune_1d(w, N, M)
    assert np.array_equal(out.contiguous().view(it).cpu().numpy(), np.where(pmask != 0, raw, 0))


def test_unaligned_packed_outputs_only():
    # aligned input, packed value arrays at a 2-byte offset (bf16): the element-wise pack kernels take over
    N, M = 2, 4
    w = _inputs("bf16", 32, 64, seed=3950)
    wd = to_dev(w)
    mask, _ = oracle.approx(w, N, M)
    md = torch.from_numpy(mask).cuda()
    vs, is_, vts, its = tm.packed_shapes(32, 64, N, M)
    bufs = [torch.zeros(vs[0] * vs[1] + 1, dtype=torch.bfloat16, device="cuda"), torch.zeros(is_[0] * is_[1] + 1, dtype=torch.uint8, device="cuda"),
            torch.zeros(vts[0] * vts[1] + 1, dtype=torch.bfloat16, device="cuda"), torch.zeros(its[0] * its[1] + 1, dtype=torch.uint8, device="cuda")]
    packed = tuple(b[1:].view(shp) for b, shp in zip(bufs, (vs, is_, vts, its)))
    assert packed[0].data_ptr() % 4 == 2
    tm.tmask_apply_pack([wd], [md], [packed], N, M)
    torch.cuda.synchronize()
    for g, t in zip(packed, oracle.apply_pack(w, mask, N, M)):
        gh = g.contiguous().view(torch.int16).cpu().numpy().view(np.uint16) if g.dtype == torch.bfloat16 else g.cpu().numpy()
        assert np.array_equal(gh.view(np.uint8), t.view(np.uint8))


# ---------------------------------------------------------------- bf16, M = 4, 8-byte aligned: narrow strips ------

@pytest.mark.parametrize("N", [1, 2, 3])
@pytest.mark.parametrize("kind,fmt,rows,cols,ld", [
    ("bf16", tm.TMASK_MASK_U8, 4, 4, 4), ("bf16", tm.TMASK_MASK_U8, 68, 132, 132), ("ties", tm.TMASK_MASK_U8, 64, 124, 124),
    ("bf16", tm.TMASK_MASK_U8, 132, 2052, 2060), ("bf16", tm.TMASK_MASK_BITS, 20, 8, 12), ("ties", tm.TMASK_MASK_BITS, 72, 264, 268)])
def test_narrow_strips(kind, fmt, rows, cols, ld, N):
    """Widths or pitches that are a multiple of four bf16 entries, not of eight: every call against the oracle, alone and
    with a matrix of the wide layout in the same batch."""
    M = 4
    w = _inputs(kind, rows, cols, seed=3960 + cols + N)
    w = w if w.dtype == np.uint16 else wl.f32_to_bf16_bits(w)
    w2 = _inputs("bf16", 16, 64, seed=3961)
    wd, wd2 = _unaligned_dev(w, ld, 0), to_dev(w2)
    ws, host = [wd, wd2], [w, w2]
    obj = torch.full((6,), -1.0, dtype=torch.float64, device="cuda")
    wsp = tm.alloc_workspace(ws, N, M)
    masks = []
    for k, fn in enumerate((tm.tmask_approx, tm.tmask_exact, tm.tmask_prune_1d)):
        masks.append([m.fill_(0xCD) for m in tm.alloc_masks(ws, fmt)])
        fn(ws, masks[-1], N, M, objective=obj[2 * k:2 * k + 2], mask_fmt=fmt, workspace=wsp)
    torch.cuda.synchronize()
    o = obj.cpu().numpy().reshape(3, 2)
    got = [[mask_to_host(m, h.shape[1], fmt) for m, h in zip(ms, host)] for ms in masks]
    for i, h in enumerate(host):
        amask, aobj = oracle.approx(h, N, M)
        _, eobj, epb = oracle.exact(h, N, M, per_block=True)
        pmask, pobj = oracle.prune_1d(h, N, M)
        assert np.array_equal(got[0][i], amask) and np.array_equal(got[2][i], pmask)
        _check_exact(h, got[1][i], N, M, epb)
        np.testing.assert_allclose(o[:, i], [aobj, eobj, pobj], rtol=1e-5)
    scores, pbs = None, [oracle.score(h, g, N, M) for h, g in zip(host, got[0])]
    sout = torch.zeros(2 * tm.SCORE_OUT_BYTES, dtype=torch.uint8, device="cuda")
    pb = torch.full((sum(h.size // 16 for h in host),), -1.0, dtype=torch.float32, device="cuda")
    tm.tmask_score(ws, masks[0], N, M, sout, per_block_obj=pb, mask_fmt=fmt, workspace=wsp)
    packed = [tm.alloc_packed(x, N, M) for x in ws]
    for pk in packed:
        for t in pk:
            t.view(torch.uint8).fill_(0xEE)
    tm.tmask_apply_pack(ws, masks[1], packed, N, M, mask_fmt=fmt)
    torch.cuda.synchronize()
    scores = tm.read_scores(sout, 2)
    np.testing.assert_allclose(pb.cpu().numpy(), np.concatenate([s.per_block.ravel() for s in pbs]), rtol=1e-5, atol=1e-30)
    for sc, so in zip(scores, pbs):
        assert (sc["kept"], sc["row_violations"], sc["col_violations"], sc["row_not_n"], sc["col_not_n"]) == \
               (so.kept, so.row_violations, so.col_violations, so.row_not_n, so.col_not_n)
        assert sc["retained_l1"] == pytest.approx(so.retained_l1, rel=1e-5)
        assert sc["total_l1"] == pytest.approx(so.total_l1, rel=1e-5)
    for pk, h, g in zip(packed, host, got[1]):
        for have, t in zip(pk, oracle.apply_pack(h, g, N, M)):
            hv = have.view(torch.int16).cpu().numpy().view(np.uint16) if have.dtype == torch.bfloat16 else have.cpu().numpy()
            assert np.array_equal(hv.view(np.uint8), t.view(np.uint8))
    # the masked copies: Algorithm 1 in place on a copy, row pruning with absorption into a padded buffer, masks written
    out = _unaligned_dev(w, ld, 0)
    dm = tm.alloc_masks([wd], fmt)
    tm.tmask_approx_dense([out], dm, [out], N, M, mask_fmt=fmt)
    out2 = torch.zeros((rows, ld), dtype=torch.bfloat16, device="cuda")[:, :cols]
    tm.tmask_prune_1d_dense([wd], None, [out2], N, M, absorb_mean=True)
    torch.cuda.synchronize()
    amask, _ = oracle.approx(w, N, M)
    assert np.array_equal(mask_to_host(dm[0], cols, fmt), amask)
    assert np.array_equal(out.contiguous().view(torch.int16).cpu().numpy().view(np.uint16), np.where(amask != 0, w, 0))
    wf = wl.bf16_bits_to_f32(w)
    want = oracle.apply_dense(wf, oracle.prune_1d(w, N, M)[0], M, absorb_mean=True)
    tol = 2.0 ** -20 * np.abs(wf.astype(np.float64)).reshape(rows, -1, M).sum(2).repeat(M, axis=1) + 2.0 ** -8 * np.abs(want)
    assert np.all(np.abs(out2.float().cpu().numpy().astype(np.float64) - want) <= tol + 1e-30)


# ---------------------------------------------------------------- batches beyond one launch ------

def test_batches_of_300_matrices_cross_the_launch_limit_and_share_index_buckets():
    # 300 matrices: more than one launch holds (256; 224 for the pack kernels), most of them one workgroup each, so many
    # matrices fall into one bucket of the coarse index and the search inside a bucket is exercised; a few larger ones
    # make the buckets uneven.  approx + exact + score + apply_pack + approx_pack + approx_dense, 2:4 fp32 and 4:8 bf16.
    rng = np.random.default_rng(4000)
    for dt, N, M in (("f32", 2, 4), ("bf16", 4, 8)):
        shapes = [(16, 16), (16, 32), (32, 16), (8 * M, 1040), (16, 64)]
        picks = rng.integers(0, len(shapes), size=300)
        picks[[7, 150, 299]] = 3
        ws = [_inputs(dt, *shapes[int(p)], seed=4100 + k) for k, p in enumerate(picks)]
        want = [oracle.approx(w, N, M) for w in ws]
        masks, obj = run_masks(tm.tmask_approx, ws, N, M)
        for k in range(300):
            assert np.array_equal(masks[k], want[k][0]), "approx, matrix %d" % k
            assert obj[k] == pytest.approx(want[k][1], rel=1e-5)
        emasks, eobj = run_masks(tm.tmask_exact, ws, N, M)
        for k in range(0, 300, 7):
            _, oobj, opb = oracle.exact(ws[k], N, M, per_block=True)
            _check_exact(ws[k], emasks[k], N, M, opb)
            assert eobj[k] == pytest.approx(oobj, rel=1e-5)
        scores, pbs = run_score(ws, masks, N, M)
        for k in range(0, 300, 5):
            o = oracle.score(ws[k], masks[k], N, M)
            assert (scores[k]["kept"], scores[k]["row_not_n"], scores[k]["col_not_n"]) == (o.kept, o.row_not_n, o.col_not_n)
            np.testing.assert_allclose(pbs[k], o.per_block, rtol=1e-5, atol=1e-30)
        packed = run_pack(ws, masks, N, M)
        fused, fmasks, fobj = run_fused(ws, N, M)
        for k in range(300):
            assert np.array_equal(fmasks[k], want[k][0]), "approx_pack, matrix %d" % k
        for k in range(0, 300, 5):
            ref = oracle.apply_pack(ws[k], masks[k], N, M)
            for g, f, t in zip(packed[k], fused[k], ref):
                assert np.array_equal(g.view(np.uint8), t.view(np.uint8)), "apply_pack, matrix %d" % k
                assert np.array_equal(f.view(np.uint8), t.view(np.uint8)), "approx_pack, matrix %d" % k
        wd = [to_dev(w) for w in ws]
        outs = [torch.empty_like(w) for w in wd]
        tm.tmask_approx_dense(wd, None, outs, N, M)
        torch.cuda.synchronize()
        it = torch.int16 if dt == "bf16" else torch.int32
        for k in range(0, 300, 5):
            raw = wd[k].view(it).cpu().numpy()
            assert np.array_equal(outs[k].view(it).cpu().numpy(), np.where(want[k][0] != 0, raw, 0)), "approx_dense, matrix %d" % k
