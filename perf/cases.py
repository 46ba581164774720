"""The work that programs have this framework do, as cases that can be timed.

A program that trains or prunes with N:M transposable masks finds masks for its layers (Algorithm 1 while it trains, the
optimal ones once for weights that are trained already), masks or compresses the weights with them, reports the quality
of a mask, and multiplies with the compressed operands in both directions.  Each operation appears at sizes from one
small layer to a whole network, for both weight types, at M = 4 ... 32, and for matrices that are no multiple of the
kernels' own tiles.

A case is a dict of plain values:
  op      "approx", "exact", "dense" (masked copy in one pass), "fused_pack" (mask and compression in one pass),
          "export" (mask, compression and score as three calls), "spmm" (product with a compressed operand)
  layers  "resnet50" (its convolutions, flattened), "bert" (its 144 linear layers), "encoder" (one of its 24 layers:
          six matrices), or "ROWSxCOLS"
  dt, N, M, bits (masks as bits instead of bytes)
  spmm:   rows x cols of the weight matrix, tokens, backward (multiply by W instead of W^T), out
"""
import math

import torch

from paper_2102_08124_amd import binding as tm
from paper_2102_08124_amd import workloads as wl

TYPES = {"f32": torch.float32, "bf16": torch.bfloat16}


def mask_case(op, layers, dt, N, M, bits=False):
    return {"op": op, "layers": layers, "dt": dt, "N": N, "M": M, "bits": bits}


def spmm_case(rows, cols, tokens, backward, out):
    return {"op": "spmm", "rows": rows, "cols": cols, "tokens": tokens, "backward": backward, "out": out}


def listed():
    return [
        # one small convolution (a 1x1 expansion of the first stage): launches and host time are all there is
        {"name": "approx_layer_f32_2of4", **mask_case("approx", "256x64", "f32", 2, 4)},
        # the mask of a whole language model extracted again during training, every layer in one call
        {"name": "approx_bert_bf16_2of4", **mask_case("approx", "bert", "bf16", 2, 4)},
        # the largest block size, for a layer-wise study of how the block size changes what a mask retains
        {"name": "approx_encoder_bf16_16of32", **mask_case("approx", "encoder", "bf16", 16, 32)},
        # what every step of dense-emulated sparse training does to its weights before the forward pass
        {"name": "dense_resnet50_f32_2of4", **mask_case("dense", "resnet50", "f32", 2, 4)},
        # optimal masks for a trained network, found once before fine-tuning
        {"name": "exact_resnet50_f32_4of8", **mask_case("exact", "resnet50", "f32", 4, 8)},
        # the same at a larger block size for one transformer layer
        {"name": "exact_encoder_bf16_8of16", **mask_case("exact", "encoder", "bf16", 8, 16)},
        # a network made ready for sparse products: mask, both compressed operands, and the report on the mask
        {"name": "export_resnet50_f32_2of4", **mask_case("export", "resnet50", "f32", 2, 4)},
        # a transformer layer compressed straight from its weights during training
        {"name": "fused_pack_encoder_bf16_4of8", **mask_case("fused_pack", "encoder", "bf16", 4, 8)},
        # a layer whose width is a multiple of four but not of eight (rows start at odd multiples of eight bytes)
        {"name": "export_ragged_bf16_2of4", **mask_case("export", "1000x2052", "bf16", 2, 4)},
        # forward product of a feed-forward layer over a training batch
        {"name": "spmm_forward_8192", **spmm_case(4096, 1024, 8192, False, "bf16")},
        # backward product of the same layer over a short, odd number of tokens, gradients in fp32
        {"name": "spmm_backward_1003", **spmm_case(4096, 1024, 1003, True, "f32")},
        # the same layer while a few sequences are decoded: the weights are read for a handful of tokens
        {"name": "spmm_decode_16", **spmm_case(4096, 1024, 16, False, "bf16")},
    ]


def _log_uniform(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _multiple(value, of, least=1):
    return max(least, round(value / of)) * of


def draw(rng):
    op = rng.choice(["approx", "exact", "dense", "fused_pack", "export", "spmm", "spmm"])
    if op == "spmm":
        tokens = max(1, int(_log_uniform(rng, 1, 8192)))
        rows = _multiple(_log_uniform(rng, 256, 4096), 64)
        cols = _multiple(_log_uniform(rng, 256, 4096), 64)
        while tokens * rows * cols > 8192 * 4096 * 1024:
            tokens //= 2
        return spmm_case(rows, cols, tokens, rng.random() < 0.5, rng.choice(["bf16", "f32"]))
    dt = rng.choice(["f32", "bf16"])
    M = {"approx": [4, 4, 8, 16, 32], "exact": [4, 8, 8, 16]}.get(op, [4, 4, 8, 16])
    M = rng.choice(M)
    N = M // 2 if rng.random() < 0.8 else rng.randrange(1, M)
    # the optimal solver's time per weight grows with M; an export passes over the weights three times
    most = {"exact": 23e6 if M <= 8 else 12.5e6, "export": 24e6}.get(op, 48e6)
    count = _log_uniform(rng, 16384, most)
    shape = _log_uniform(rng, 0.25, 4.0)                     # rows : cols
    rows = _multiple(math.sqrt(count * shape), M)
    unit = M if rng.random() < 0.25 else max(M, 64)          # a quarter of the widths are as odd as M allows
    cols = _multiple(min(count / rows, most / rows), unit)
    bits = cols % 64 == 0 and rng.random() < 0.25
    return mask_case(op, "%dx%d" % (rows, cols), dt, N, M, bits)


def shapes(case):
    text = case["layers"]
    if text == "resnet50":
        return wl.resnet50_conv_shapes()
    if text == "bert":
        return wl.bert_large_linear_shapes()
    if text == "encoder":
        return wl.bert_large_linear_shapes()[:6]
    rows, cols = text.split("x")
    return [(int(rows), int(cols))]


def _weights(case, seed):
    """Weights as a network is initialised: normal, fan-out scaled for convolutions, 0.02 for the linear layers."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    out = []
    for shape in shapes(case):
        std = math.sqrt(2.0 / (shape[0] * wl.resnet50_kernel_area(shape))) if case["layers"] == "resnet50" else 0.02
        out.append((torch.randn(shape, device="cuda", generator=gen) * std).to(TYPES[case["dt"]]))
    return out


def _product_inputs(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    w = (torch.randn((case["rows"], case["cols"]), device="cuda", generator=gen) * 0.02).to(torch.bfloat16)
    width = case["rows"] if case["backward"] else case["cols"]
    x = torch.randn((case["tokens"], width), device="cuda", generator=gen).to(torch.bfloat16)
    return w, x


def _flat(shape_lists, dtypes):
    """One buffer per kind of output for the whole network, and every matrix's views of them (a program that keeps its
    masks or compressed weights for a checkpoint or a collective allocates them like this)."""
    flats = [torch.empty(sum(r * c for r, c in shapes_), dtype=dt, device="cuda")
             for shapes_, dt in zip(shape_lists, dtypes)]
    views = []
    for flat, shapes_ in zip(flats, shape_lists):
        parts = torch.split(flat, [r * c for r, c in shapes_])
        views.append([p.view(shape) for p, shape in zip(parts, shapes_)])
    return flats, list(zip(*views))


def _flat_masks(ws, fmt):
    (flat,), views = _flat([[tm.mask_shape(w.shape[0], w.shape[1], fmt) for w in ws]], [torch.uint8])
    return flat, [v[0] for v in views]


def _flat_packed(ws, N, M):
    kinds = list(zip(*[tm.packed_shapes(w.shape[0], w.shape[1], N, M) for w in ws]))
    return _flat(kinds, [ws[0].dtype, torch.uint8, ws[0].dtype, torch.uint8])


def prepare(case, seed):
    state = {"case": case}
    if case["op"] == "spmm":
        w, x = _product_inputs(case, seed)
        packed = tm.alloc_packed(w, 2, 4)
        tm.tmask_approx_pack([w], None, [packed], 2, 4)
        rows, cols = case["rows"], case["cols"]
        if case["backward"]:
            operand = (packed[2], packed[3], cols, rows)
        else:
            operand = (packed[0], packed[1], rows, cols)
        y = torch.empty((case["tokens"], operand[2]), dtype=TYPES[case["out"]], device="cuda")
        state.update(operand=operand, x=x, y=y)
        return state
    op, N, M = case["op"], case["N"], case["M"]
    ws = _weights(case, seed)
    fmt = tm.TMASK_MASK_BITS if case["bits"] else tm.TMASK_MASK_U8
    state.update(ws=ws, fmt=fmt)
    if op == "dense":
        (flat,), views = _flat([[tuple(w.shape) for w in ws]], [ws[0].dtype])
        state.update(out=flat, batch=tm.DenseBatch(ws, None, [v[0] for v in views]))
        return state
    state["workspace"] = tm.alloc_workspace(ws, N, M)
    state["objective"] = torch.zeros(len(ws), dtype=torch.float64, device="cuda")
    if op in ("fused_pack", "export"):
        state["packed"], packed = _flat_packed(ws, N, M)
    if op == "fused_pack":
        # the one-pass kernels need no mask; the other N:M go through one
        state["masks"], masks = (None, None) if (N, M) in ((2, 4), (4, 8)) else _flat_masks(ws, fmt)
        state["batch"] = tm.FusedBatch(ws, masks, packed, N, M, state["objective"])
        return state
    state["masks"], masks = _flat_masks(ws, fmt)
    state.update(batch=tm.MatBatch(ws, masks, state["objective"]))
    if op == "export":
        state["pack_batch"] = tm.PackBatch(ws, masks, packed, N, M)
        out = torch.zeros(len(ws) * tm.SCORE_OUT_BYTES, dtype=torch.uint8, device="cuda")
        blocks = sum(w.numel() for w in ws) // (M * M)
        state.update(score=out, per_block=torch.empty(blocks, dtype=torch.float32, device="cuda"),
                     sums=out.view(torch.float64).view(len(ws), 7)[:, :2],
                     counts=out.view(torch.int64).view(len(ws), 7)[:, 2:])
    return state


def run(state):
    case = state["case"]
    op = case["op"]
    if op == "spmm":
        vals, idx, rows, cols = state["operand"]
        tm.tmask_spmm24(vals, idx, rows, cols, state["x"], state["y"])
        return state["y"]
    N, M, fmt = case["N"], case["M"], state["fmt"]
    if op == "dense":
        tm.tmask_approx_dense(state["batch"], None, None, N, M, mask_fmt=fmt)
        return state["out"]
    workspace = state["workspace"]
    if op == "fused_pack":
        tm.tmask_approx_pack(state["batch"], None, None, N, M, mask_fmt=fmt, workspace=workspace)
        result = {"objective": state["objective"], "packed": state["packed"]}
        return result if state["masks"] is None else {**result, "masks": state["masks"]}
    find = tm.tmask_exact if op == "exact" else tm.tmask_approx
    find(state["batch"], None, N, M, mask_fmt=fmt, workspace=workspace)
    result = {"objective": state["objective"], "masks": state["masks"]}
    if op == "export":
        tm.tmask_apply_pack(state["pack_batch"], None, None, N, M, mask_fmt=fmt, workspace=workspace)
        tm.tmask_score(state["batch"], None, N, M, state["score"], per_block_obj=state["per_block"], mask_fmt=fmt,
                       workspace=workspace)
        result.update(packed=state["packed"], sums=state["sums"], counts=state["counts"], per_block=state["per_block"])
    return result


def work(case):
    if case["op"] == "spmm":
        rows, cols, tokens = case["rows"], case["cols"], case["tokens"]
        outs, ins = (cols, rows) if case["backward"] else (rows, cols)
        out_bytes = 4 if case["out"] == "f32" else 2
        # the compressed operand (half the values in two bytes, two bits of position each), x and y; kept products
        return {"bytes": rows * cols + rows * cols // 8 + tokens * (2 * ins + out_bytes * outs),
                "flops": tokens * rows * cols}
    op, N, M = case["op"], case["N"], case["M"]
    count = sum(r * c for r, c in shapes(case))
    size = 4 if case["dt"] == "f32" else 2
    mask = 0.125 if case["bits"] else 1.0
    packed = 2 * (N / M) * (size + (M - 1).bit_length() / 8)     # values and positions, for W and for W^T
    if op in ("approx", "exact"):
        per = size + mask
    elif op == "dense":
        per = 2 * size
    elif op == "fused_pack":
        per = size + packed + (0.0 if (N, M) in ((2, 4), (4, 8)) else mask)
    else:                                                        # export: each call reads and writes what it is given
        per = (size + mask) + (size + mask + packed) + (size + mask + 4 / M ** 2)
    return {"bytes": int(count * per), "flops": 0}


def tolerance(case):
    """About four times what was measured between the path and a correct one that sums in another order."""
    op = case["op"]
    if op == "spmm":
        if case["out"] == "bf16":
            # against the 64-bit product rounded to bf16: 3e-5, single results one unit in the last place (2^-7) apart
            return {"rel": 1.2e-4, "max": 1.6e-2}
        return {"rel": 8e-7, "max": 1e-5}                        # against the 64-bit product: 2e-7, 2.3e-6
    if op == "dense":
        return "exact"
    if op == "exact":
        # Different masks of a block can be equally good, in bf16 above all; they retain the same.  The masks of W^T,
        # transposed, against those of W: up to 6.5e-4 of the entries differ in bf16, none in fp32; objectives 5e-9.
        return {"rel": 2e-8, "max": 2e-7, "differ": 2.6e-3 if case["dt"] == "bf16" else 1e-5}
    # masks, positions and counts are whole numbers, packed values are copies; sums (per block in fp32, 4e-8; whole ones
    # in fp64 over fp32 strips, 1e-8) may be taken in another order
    return {"rel": 2e-7, "max": 1e-6}


def _reference_mask(w, N, M):
    """Algorithm 1 in its rank form: an entry stays iff M - N entries of its row and of its column precede it."""
    rows, cols = w.shape
    a = w.abs().double().view(rows // M, M, cols // M, M)
    keep = torch.ones(a.shape, dtype=torch.bool, device=w.device)
    for dim in (1, 3):
        order = torch.sort(a, dim=dim, stable=True).indices
        light = order.narrow(dim, 0, M - N)
        keep.scatter_(dim, light, False)
    return keep.view(rows, cols)


def _patterns4(N):
    """All 4 x 4 patterns with N kept in every row and column, one a row of sixteen."""
    lines = [b for b in range(16) if bin(b).count("1") == N]
    found = []
    for r0 in lines:
        for r1 in lines:
            for r2 in lines:
                for r3 in lines:
                    rows = (r0, r1, r2, r3)
                    if all(sum(r >> c & 1 for r in rows) == N for c in range(4)):
                        found.append([r >> c & 1 for r in rows for c in range(4)])
    return found


def exact(case, seed):
    if case["op"] == "spmm":
        w, x = _product_inputs(case, seed)
        w = w.double() * _reference_mask(w, 2, 4)
        return x.double() @ (w if case["backward"] else w.t())
    op, N, M = case["op"], case["N"], case["M"]
    ws = _weights(case, seed)
    if op == "exact":
        if M != 4:
            return None
        pats = torch.tensor(_patterns4(N), dtype=torch.float64, device="cuda")
        best = []
        for w in ws:
            blocks = w.abs().double().view(w.shape[0] // 4, 4, w.shape[1] // 4, 4).permute(0, 2, 1, 3).reshape(-1, 16)
            best.append((blocks @ pats.t()).max(dim=1).values.sum())
        return {"objective": torch.stack(best), "masks": None}
    keeps = [_reference_mask(w, N, M) for w in ws]
    if op == "dense":
        return torch.cat([(w.double() * k).flatten() for w, k in zip(ws, keeps)])
    kept = [w.abs().double() * k for w, k in zip(ws, keeps)]
    objective = torch.stack([k.sum() for k in kept])
    masks = None if case["bits"] else torch.cat([k.flatten().to(torch.uint8) for k in keeps])
    if op == "fused_pack":
        result = {"objective": objective, "packed": [None] * 4}
        return result if (N, M) in ((2, 4), (4, 8)) else {**result, "masks": masks}
    result = {"objective": objective, "masks": masks}
    if op == "export":
        total = torch.stack([w.abs().double().sum() for w in ws])
        per = [k.view(k.shape[0] // M, M, k.shape[1] // M, M).sum(dim=(1, 3)).flatten() for k in kept]
        result.update(packed=[None] * 4, sums=torch.stack([objective, total], dim=1), counts=None,
                      per_block=torch.cat(per))
    return result
