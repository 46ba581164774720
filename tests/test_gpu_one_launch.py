"""Objectives and scores that a launch adds up itself: the last workgroup of a matrix waits for the partial results of the others,
which carry the tags of their launch.  Whatever the workspace holds before a call, and however often a captured call is replayed,
the sums are those of the masks; the objective has the bits of tmask_approx_noalloc, which adds them up in a second launch."""
import ctypes

import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2102_08124_amd import binding as tm   # noqa: E402

F32, BF16 = torch.float32, torch.bfloat16


def _weights(shapes, dtype, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    return [torch.randn(s, device="cuda", generator=gen).to(dtype) for s in shapes]


def _garbage(wsp, kind):
    words = wsp[:wsp.numel() // 4 * 4].view(torch.int32)
    if kind == "random":
        words.random_(-2 ** 31, 2 ** 31 - 1)
    else:
        words.fill_(kind)


def _kept(ws, masks):
    return torch.stack([(w.double().abs() * (m != 0)).sum() for w, m in zip(ws, masks)])


# workgroups of a matrix: 256 strips of 16 bytes x M rows each at M <= 16 aligned (fp32 2:4: 4096 weights), tiles of 32 x 64 at M = 32
# (bf16 16:32: four of them), 64 columns x M rows on unaligned matrices.  One, two, 256 and 257 that report to a last one, the most
# that do (8 for each thread of it) and one more, more matrices than may wait in a launch, ragged ends.
CASES = [
    ([(64, 64)], F32, 2, 4), ([(4, 8)], F32, 1, 4), ([(64, 128)], F32, 3, 4), ([(1024, 1024), (64, 72), (1028, 1024)], F32, 2, 4),
    ([(2048, 4096)], F32, 2, 4), ([(2052, 4096)], F32, 2, 4), ([(1024, 1024)] * 32, F32, 2, 4), ([(1024, 1024)] * 33, F32, 2, 4),
    ([(1000, 2052)], BF16, 2, 4), ([(1024, 2048), (8, 16)], BF16, 4, 8), ([(1024, 1040)], F32, 4, 8), ([(512, 528)], BF16, 8, 16),
    ([(512, 512)], F32, 5, 16), ([(1024, 1024), (32, 32)], BF16, 16, 32), ([(256, 4160)], F32, 16, 32), ([(1024, 1056)], F32, 16, 32),
    ([(256, 516)], BF16, 1, 4), ([(64, 68)], BF16, 1, 4),
    ([(2048, 4096)] * 7, F32, 2, 4),
    # a score adds up 256 workgroups itself and no more: strips, narrow strips, columns
    ([(1024, 1024)], F32, 2, 4), ([(1024, 1024), (4, 8)], F32, 2, 4), ([(512, 2044)], BF16, 2, 4), ([(512, 2044), (4, 4)], BF16, 2, 4),
    ([(512, 1024)], BF16, 16, 32), ([(512, 1024), (32, 32)], BF16, 16, 32), ([(256, 512)], F32, 16, 32), ([(64, 64)], F32, 8, 32)]


@pytest.mark.parametrize("shapes,dtype,N,M", CASES)
def test_objectives(shapes, dtype, N, M):
    ws = _weights(shapes, dtype, 11 * N + M)
    wsp = tm.alloc_workspace(ws, N, M)
    masks = tm.alloc_masks(ws)
    obj, ref = torch.zeros(len(ws), dtype=torch.float64, device="cuda"), torch.zeros(len(ws), dtype=torch.float64, device="cuda")
    tm.tmask_approx_noalloc(ws, masks, N, M, objective=ref)
    for find in (tm.tmask_approx, tm.tmask_exact if M <= 16 else tm.tmask_approx, tm.tmask_prune_1d):
        got = []
        for kind in ("random", 0, -1, 0x3F800000):
            _garbage(wsp, kind)
            obj.fill_(-1.0)
            find(ws, masks, N, M, objective=obj, workspace=wsp)
            torch.cuda.synchronize()
            got.append(obj.clone())
        # fp32 sums of at most 128 terms inside a lane and 64 lanes
        assert torch.allclose(got[0], _kept(ws, masks), rtol=2e-5, atol=0.0)
        assert all(torch.equal(got[0], g) for g in got)
        if find is tm.tmask_approx:
            assert torch.equal(got[0], ref)


@pytest.mark.parametrize("shapes,dtype,N,M", CASES)
def test_scores(shapes, dtype, N, M):
    ws = _weights(shapes, dtype, 13 * N + M)
    wsp = tm.alloc_workspace(ws, N, M)
    masks = tm.alloc_masks(ws)
    for m in masks:
        m.random_(0, 2)
    out = torch.zeros(len(ws) * tm.SCORE_OUT_BYTES, dtype=torch.uint8, device="cuda")
    got = []
    for kind in ("random", 0, -1):
        _garbage(wsp, kind)
        out.fill_(0xA5)
        tm.tmask_score(ws, masks, N, M, out, workspace=wsp)
        torch.cuda.synchronize()
        got.append(out.clone())
    assert torch.equal(got[0], got[1]) and torch.equal(got[0], got[2])
    for w, m, s in zip(ws, masks, tm.read_scores(out, len(ws))):
        r, c = w.shape
        rows = (m != 0).view(r, c // M, M).sum(2)
        cols = (m != 0).view(r // M, M, c).sum(1)
        assert s["kept"] == int((m != 0).sum())
        assert (s["row_violations"], s["row_not_n"]) == (int((rows > N).sum()), int((rows != N).sum()))
        assert (s["col_violations"], s["col_not_n"]) == (int((cols > N).sum()), int((cols != N).sum()))
        assert s["total_l1"] == pytest.approx(float(w.double().abs().sum()), rel=2e-5)
        assert s["retained_l1"] == pytest.approx(float((w.double().abs() * (m != 0)).sum()), rel=2e-5)


@pytest.mark.parametrize("dtype,N,M", [(F32, 2, 4), (BF16, 4, 8), (F32, 4, 8)])
def test_one_pass_with_a_small_workspace(dtype, N, M):
    """tmask_approx_pack takes a workspace of 8 bytes per tile, too small for records of 16: then by two launches."""
    ws = _weights([(1024, 1024), (64, 264)], dtype, 17)
    packed = [tm.alloc_packed(w, N, M) for w in ws]
    ref = torch.zeros(2, dtype=torch.float64, device="cuda")
    tm.tmask_approx(ws, tm.alloc_masks(ws), N, M, objective=ref, workspace=tm.alloc_workspace(ws, N, M))
    batch = tm.FusedBatch(ws, None, packed, N, M, ref.clone())
    full = tm.alloc_workspace(ws, N, M)
    got = []
    for size in (full.numel(), 8 * (16 * 16 + 2), 8 * (8 * 4 + 4)):
        _garbage(full, "random")
        batch.objective.fill_(-1.0)
        rc = tm.load_library().tmask_approx_pack(batch.arr, 2, batch.dt, N, M, tm.TMASK_MASK_U8, ctypes.c_void_p(full.data_ptr()), size,
                                                 ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
        torch.cuda.synchronize()
        if rc == tm.TMASK_OK:
            got.append(batch.objective.clone())
        else:
            assert rc == tm.TMASK_ERR_WORKSPACE and size < full.numel()
    assert len(got) >= 2
    for g in got:
        assert torch.allclose(g, ref, rtol=2e-6, atol=0.0)


@pytest.mark.parametrize("shape,dtype,N,M", [((256, 256), F32, 2, 4), ((256, 256), F32, 1, 4), ((256, 256), F32, 4, 8), ((256, 256), BF16, 4, 8),
                                             ((256, 256), BF16, 8, 16), ((256, 512), F32, 5, 16), ((64, 256), BF16, 16, 32),
                                             ((64, 256), F32, 16, 32), ((256, 516), BF16, 1, 4)])
@pytest.mark.parametrize("n,few", [(7, True), (8, False)])
def test_how_many_matrices_a_launch_adds_up(shape, dtype, N, M, n, few):
    """Seven waiting workgroups to a launch.  The workspace shows which way a call went: what a launch hands over to itself it
    clears, what it leaves for a second launch stays."""
    ws = _weights([shape] * n, dtype, 31)
    masks, wsp = tm.alloc_masks(ws), tm.alloc_workspace(ws, N, M)
    obj = torch.zeros(n, dtype=torch.float64, device="cuda")
    out = torch.zeros(n * tm.SCORE_OUT_BYTES, dtype=torch.uint8, device="cuda")
    calls = [(lambda f=f: f(ws, masks, N, M, objective=obj, workspace=wsp)) for f in (tm.tmask_approx, tm.tmask_exact, tm.tmask_prune_1d)]
    if 2 * N == M <= 8:
        packed = [tm.alloc_packed(w, N, M) for w in ws]
        calls.append(lambda: tm.tmask_approx_pack(ws, masks, packed, N, M, objective=obj, workspace=wsp))
    for k, call in enumerate(calls):
        wsp.zero_()
        obj.fill_(-1.0)
        call()
        torch.cuda.synchronize()
        assert bool(wsp.any()) != few, k
        assert torch.allclose(obj, _kept(ws, masks), rtol=2e-5, atol=0.0)
    wsp.zero_()
    tm.tmask_score(ws, masks, N, M, out, workspace=wsp)
    torch.cuda.synchronize()
    assert bool(wsp.any()) != few
    assert [s["kept"] for s in tm.read_scores(out, n)] == [int((m != 0).sum()) for m in masks]


@pytest.mark.parametrize("n", [8, 9, 40, 224, 230])
@pytest.mark.parametrize("dtype,N,M", [(F32, 2, 4), (BF16, 4, 8)])
def test_one_pass_over_many_small_matrices(dtype, N, M, n):
    """One launch has room for the objectives of eight; the rest take the second launch, also past the 224 of a launch."""
    ws = _weights([(16, 64)] * n, dtype, 37)
    packed = [tm.alloc_packed(w, N, M) for w in ws]
    obj, ref = torch.full((n,), -1.0, dtype=torch.float64, device="cuda"), torch.zeros(n, dtype=torch.float64, device="cuda")
    wsp = tm.alloc_workspace(ws, N, M)
    tm.tmask_approx_noalloc(ws, tm.alloc_masks(ws), N, M, objective=ref)
    _garbage(wsp, "random")
    tm.tmask_approx_pack(ws, None, packed, N, M, objective=obj, workspace=wsp)
    torch.cuda.synchronize()
    assert torch.allclose(obj, ref, rtol=2e-6, atol=0.0)


# the call, the matrices and, for each of these, the workgroups: workgroup 0 .. n - 2 of a matrix leave records of so many words
REPLAYS = [("approx", [(1024, 1024), (520, 136)], F32, 4, 8, 2, [128, 9]), ("exact", [(512, 512), (264, 136)], BF16, 4, 8, 2, [32, 5]),
           ("approx", [(1024, 1024)], BF16, 16, 32, 2, [128]), ("approx", [(256, 512)], F32, 5, 16, 2, [8]), ("prune", [(256, 256)], F32, 2, 4, 2, [16]),
           ("pack", [(1024, 1024)], F32, 4, 8, 2, None), ("score", [(512, 512), (136, 264)], F32, 2, 4, 7, [64, 9]), ("score", [(256, 256)], F32, 16, 32, 7, [32]),
           ("score", [(256, 516)], BF16, 2, 4, 7, [33])]


@pytest.mark.parametrize("kind,shapes,dtype,N,M,words,workgroups", REPLAYS)
def test_a_replay_finds_nothing_of_the_one_before(kind, shapes, dtype, N, M, words, workgroups):
    """One call in a graph, replayed with other weights and nothing else in its workspace in between: records that the last replay
    left would bear this one's tags, and their sums would be the last weights'.  References come from a second workspace."""
    ws = _weights(shapes, dtype, 19)
    masks, wsp, other = tm.alloc_masks(ws), tm.alloc_workspace(ws, N, M).zero_(), tm.alloc_workspace(ws, N, M)
    packed = [tm.alloc_packed(w, N, M) for w in ws] if kind == "pack" else None
    obj = torch.zeros(len(ws), dtype=torch.float64, device="cuda")
    out = torch.zeros(len(ws) * tm.SCORE_OUT_BYTES, dtype=torch.uint8, device="cuda")
    for m in masks:
        m.random_(0, 2)

    def call(space):
        if kind == "score":
            tm.tmask_score(ws, masks, N, M, out, workspace=space)
        elif kind == "pack":
            tm.tmask_approx_pack(ws, None, packed, N, M, objective=obj, workspace=space)
        else:
            {"approx": tm.tmask_approx, "exact": tm.tmask_exact, "prune": tm.tmask_prune_1d}[kind](ws, masks, N, M, objective=obj, workspace=space)

    call(other)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=torch.cuda.Stream()):
        call(wsp)
    seen = []
    for turn in range(6):
        for w in ws:
            w.mul_(1.25 if turn % 3 else -0.5)
        call(other)
        torch.cuda.synchronize()
        want = (obj.clone(), out.clone())
        obj.fill_(-1.0)
        out.fill_(0xA5 if kind == "score" else 0)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(obj if kind != "score" else out, want[kind == "score"]), turn
        seen.append(want[kind == "score"])
        assert not bool(wsp.any())                             # one launch, and no record left
    assert all(not torch.equal(a, b) for a, b in zip(seen, seen[1:]))


@pytest.mark.parametrize("kind,shapes,dtype,N,M,words,workgroups", [r for r in REPLAYS if r[6] is not None])
def test_records_are_cleared_where_they_lie(kind, shapes, dtype, N, M, words, workgroups):
    """Of a workspace full of ones, a call changes the words of its records, to zero, and no others (the last workgroup of a matrix has
    no record)."""
    ws = _weights(shapes, dtype, 41)
    masks, wsp = tm.alloc_masks(ws), tm.alloc_workspace(ws, N, M)
    wsp.fill_(0xFF)
    obj = torch.zeros(len(ws), dtype=torch.float64, device="cuda")
    if kind == "score":
        for m in masks:
            m.fill_(1)
        tm.tmask_score(ws, masks, N, M, torch.zeros(len(ws) * tm.SCORE_OUT_BYTES, dtype=torch.uint8, device="cuda"), workspace=wsp)
    else:
        {"approx": tm.tmask_approx, "exact": tm.tmask_exact, "prune": tm.tmask_prune_1d}[kind](ws, masks, N, M, objective=obj, workspace=wsp)
    torch.cuda.synchronize()
    want = [-1] * (wsp.numel() // 8)
    first = 0
    for n in workgroups:
        want[words * first:words * (first + n - 1)] = [0] * (words * (n - 1))
        first += n
    assert wsp[:len(want) * 8].view(torch.int64).tolist() == want


def test_replays_with_anything_in_the_workspace_between():
    """Several calls in a graph share a workspace, which eager calls use, and which is overwritten, between the replays."""
    shapes = [(1024, 1024), (520, 136)]
    ws = _weights(shapes, F32, 19)
    masks, wsp = tm.alloc_masks(ws), tm.alloc_workspace(ws, 4, 8)
    packed = [tm.alloc_packed(w, 4, 8) for w in ws]
    obj = torch.zeros(6, dtype=torch.float64, device="cuda")
    out = torch.zeros(2 * tm.SCORE_OUT_BYTES, dtype=torch.uint8, device="cuda")

    def calls():
        tm.tmask_exact(ws, masks, 4, 8, objective=obj[:2], workspace=wsp)
        tm.tmask_score(ws, masks, 4, 8, out, workspace=wsp)
        tm.tmask_approx(ws, masks, 4, 8, objective=obj[2:4], workspace=wsp)
        tm.tmask_approx_pack(ws, None, packed, 4, 8, objective=obj[4:], workspace=wsp)

    calls()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    side = torch.cuda.Stream()
    with torch.cuda.graph(graph, stream=side):
        calls()
    for turn in range(6):
        for w in ws:
            w.mul_(1.25)
        calls()
        torch.cuda.synchronize()
        want, score = obj.clone(), out.clone()
        if turn % 2:
            _garbage(wsp, "random" if turn % 4 == 1 else 0)
        obj.fill_(-1.0)
        out.fill_(0)
        graph.replay()
        if turn == 4:                              # twice in a row
            graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(obj, want) and torch.equal(out, score)


def test_calls_side_by_side_on_two_streams():
    ws = [_weights([(1024, 1024)] * 3, F32, 23 + k) for k in range(2)]
    masks = [tm.alloc_masks(w) for w in ws]
    wsp = [tm.alloc_workspace(w, 2, 4) for w in ws]
    obj = [torch.zeros(3, dtype=torch.float64, device="cuda") for _ in ws]
    want = []
    for k in range(2):
        tm.tmask_approx(ws[k], masks[k], 2, 4, objective=obj[k], workspace=wsp[k])
        torch.cuda.synchronize()
        want.append(obj[k].clone())
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    batches = [tm.MatBatch(ws[k], masks[k], obj[k]) for k in range(2)]
    for _ in range(50):
        for k in range(2):
            tm.tmask_approx(batches[k], None, 2, 4, workspace=wsp[k], stream=streams[k])
    torch.cuda.synchronize()
    assert torch.equal(obj[0], want[0]) and torch.equal(obj[1], want[1])


def test_matrices_without_an_objective_between_others():
    ws = _weights([(1024, 512), (512, 512), (1024, 1024)], F32, 29)
    masks = tm.alloc_masks(ws)
    obj = torch.full((3,), -1.0, dtype=torch.float64, device="cuda")
    batch = tm.MatBatch(ws, masks, obj)
    batch.arr[1].objective = None
    tm.tmask_approx(batch, None, 4, 8, workspace=tm.alloc_workspace(ws, 4, 8))
    torch.cuda.synchronize()
    want = _kept(ws, masks)
    assert float(obj[1]) == -1.0
    assert torch.allclose(obj[[0, 2]], want[[0, 2]], rtol=2e-6, atol=0.0)


@pytest.mark.parametrize("shapes,dtype,N,M,itself", [([(1024, 1024)], F32, 2, 4, True), ([(1024, 1024), (4, 8)], F32, 2, 4, False),
                                                     ([(512, 2044)], BF16, 2, 4, True), ([(512, 2044), (4, 4)], BF16, 2, 4, False),
                                                     ([(512, 1024)], BF16, 16, 32, True), ([(512, 1024), (32, 32)], BF16, 16, 32, False)])
def test_a_score_of_256_workgroups_is_one_launch_and_of_257_two(shapes, dtype, N, M, itself):
    ws = _weights(shapes, dtype, 43)
    masks, wsp = tm.alloc_masks(ws), tm.alloc_workspace(ws, N, M).zero_()
    for m in masks:
        m.fill_(1)
    tm.tmask_score(ws, masks, N, M, torch.zeros(len(ws) * tm.SCORE_OUT_BYTES, dtype=torch.uint8, device="cuda"), workspace=wsp)
    torch.cuda.synchronize()
    assert bool(wsp.any()) != itself
