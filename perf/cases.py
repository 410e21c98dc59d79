"""The work that a user of this package has it do, as cases that can be timed and compared.

Four kinds, all through the package's public entry points: the forward pass of one condensed layer, the forward pass of an
MLP block whose second layer reads only the first one's stored neurons, condensing a trained layer (dense weight and mask
in, condensed layer out), and one connectivity update during training.  Shapes are those of the package's configurations
(the 768 <-> 3072 projections of a ViT-B/16 block at 80-99 % sparsity, the 4096 -> 16384 bf16 layer) and ragged ones
between and below them; topologies are random constant fan-in masks, weights N(0, 1/K), activations N(0, 1).
"""
from __future__ import annotations

import math

import torch

from paper_2305_02299_amd import CondensedLinear, condense_layer, fold_mlp
from paper_2305_02299_amd import binding as B_

# Upper ends of what draw() gives: multiply-adds of a forward pass, elements of a weight matrix.  The largest listed
# cases (4096 -> 16384 at batch 2048, and its 67 million weights) lie above both.
MAX_TERMS = 4_000_000_000
MAX_CONDENSE = 32_000_000
MAX_UPDATE = 8_000_000


def _forward(d_in, d_out, sparsity, batch, dtype="f32", ablated=0, indices="uniform", form="condensed", narrow=False):
    return {"kind": "forward", "d_in": d_in, "d_out": d_out, "sparsity": sparsity, "batch": batch, "dtype": dtype, "ablated": ablated,
            "indices": indices, "form": form, "narrow": narrow}


def _mlp(d_model, d_hidden, sparsity, batch, ablated):
    return {"kind": "mlp", "d_in": d_model, "d_out": d_hidden, "sparsity": sparsity, "batch": batch, "ablated": ablated, "dtype": "f32"}


def _condense(d_in, d_out, sparsity, dtype="f32", ablated=0):
    return {"kind": "condense", "d_in": d_in, "d_out": d_out, "sparsity": sparsity, "dtype": dtype, "ablated": ablated}


def _update(d_in, d_out, sparsity, ablated, moved):
    return {"kind": "update", "d_in": d_in, "d_out": d_out, "sparsity": sparsity, "ablated": ablated, "moved": moved, "dtype": "f32"}


def listed():
    return [
        # Online inference, one sample at a time through the up-projection of a ViT-B/16 block: the smallest call.
        dict(_forward(768, 3072, 90, 1), name="online_768x3072"),
        # Online inference through the large layer with bf16 weights and 16-bit indices: the weights have to be streamed.
        dict(_forward(4096, 16384, 95, 1, "bf16", 20, "clustered", narrow=True), name="online_4096x16384_bf16"),
        # A small serving batch through the down-projection, 30 % of its neurons ablated.
        dict(_forward(3072, 768, 90, 16, ablated=30), name="serve16_3072x768"),
        # A ragged layer and batch: nothing is a multiple of a tile, rows are not 16-byte aligned.
        dict(_forward(1000, 777, 95, 37, ablated=10), name="ragged_1000x777"),
        # The headline benchmark: the up-projection at 90 % sparsity and batch 256.
        dict(_forward(768, 3072, 90, 256), name="batch256_768x3072"),
        # Modest sparsity at a throughput batch, with the form of the layer left to the library.
        dict(_forward(768, 3072, 80, 1024, form="auto"), name="batch1024_768x3072_auto"),
        # The large bf16 layer at batch 2048 with clustered indices, in condensed form.
        dict(_forward(4096, 16384, 95, 2048, "bf16", 20, "clustered"), name="batch2048_4096x16384_bf16"),
        # The same layer with the form left to the library.
        dict(_forward(4096, 16384, 95, 2048, "bf16", 20, "clustered", form="auto"), name="batch2048_4096x16384_auto"),
        # An MLP block (linear, GELU, linear) whose hidden width is reduced by ablation.
        dict(_mlp(768, 3072, 90, 256, 30), name="mlp256_768_3072"),
        # Condensing a trained layer for deployment: a ViT projection, and the large layer.
        dict(_condense(768, 3072, 90), name="condense_768x3072"),
        dict(_condense(4096, 16384, 95, "bf16", 20), name="condense_4096x16384_bf16"),
        # One connectivity update of a ViT projection during training, 30 % of the weights moved.
        dict(_update(768, 3072, 90, 0, 30), name="update_768x3072"),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, round(math.exp(rng.uniform(math.log(lo), math.log(hi + 0.49))))))


def _width(rng, lo, hi):
    """Widths over the logarithm of the range: two of three a multiple of 64 as in trained models, the others any number."""
    n = _log_int(rng, lo, hi)
    return n if rng.random() < 1 / 3 or n < 64 else (n + 32) // 64 * 64


def draw(rng):
    kind = rng.choice(["forward"] * 6 + ["mlp", "condense", "update"])
    ablated = rng.choice([0, rng.randint(1, 50)])
    sparsity = rng.randint(80, 99)
    while True:
        if kind == "forward":
            c = _forward(_width(rng, 100, 4096), _width(rng, 100, 16384), sparsity, _log_int(rng, 1, 2048), rng.choice(["f32", "bf16"]), ablated,
                         rng.choice(["uniform", "clustered"]), rng.choice(["condensed", "condensed", "auto"]), False)
            # 16-bit indices are read by the condensed form; the structured form keeps no indices
            c["narrow"] = c["form"] == "condensed" and rng.random() < 1 / 3
            fits = _stored(c) * _fan_in(c) * c["batch"] <= MAX_TERMS
        elif kind == "mlp":
            d_model = _width(rng, 100, 1024)
            c = _mlp(d_model, rng.choice([2, 3, 4]) * d_model, sparsity, _log_int(rng, 1, 1024), ablated)
            fits = True
        elif kind == "condense":
            c = _condense(_width(rng, 100, 4096), _width(rng, 100, 16384), sparsity, rng.choice(["f32", "bf16"]), ablated)
            fits = c["d_in"] * c["d_out"] <= MAX_CONDENSE
        else:
            c = _update(_width(rng, 100, 4096), _width(rng, 100, 4096), sparsity, ablated, rng.randint(5, 30))
            fits = c["d_in"] * c["d_out"] <= MAX_UPDATE
        if fits:
            return c


def _fan_in(case, d_in=None):
    return ((d_in or case["d_in"]) * (100 - case["sparsity"]) + 99) // 100


def _stored(case):
    return case["d_out"] - case["d_out"] * case["ablated"] // 100


def _dtype(case):
    return torch.float32 if case["dtype"] == "f32" else torch.bfloat16


def _mask(gen, d_in, d_out, K, n_stored, clustered=False):
    """A constant fan-in mask: n_stored rows hold K ones, the others none.  Clustered: half of a row's ones lie in one window of 512 columns."""
    column = torch.arange(d_in, dtype=torch.int32, device="cuda")
    key = (torch.randint(0, 1 << 19, (d_out, d_in), dtype=torch.int32, device="cuda", generator=gen) << 12) + column  # no two keys of a row are equal
    mask = torch.zeros((d_out, d_in), dtype=torch.uint8, device="cuda")
    left = K
    if clustered and d_in > 512:
        start = torch.randint(0, d_in - 512 + 1, (d_out, 1), dtype=torch.int32, device="cuda", generator=gen)
        inside = (column >= start) & (column < start + 512)
        if min(K // 2, 512):
            mask.scatter_(1, torch.where(inside, key, -1).topk(min(K // 2, 512), dim=1).indices, 1)
        left -= min(K // 2, 512)
    mask.scatter_(1, torch.where(mask > 0, -1, key).topk(left, dim=1).indices, 1)
    mask[torch.randperm(d_out, device="cuda", generator=gen)[n_stored:]] = 0
    return mask


def _normal(gen, shape, std, dtype=torch.float32):
    return (torch.randn(shape, device="cuda", generator=gen) * std).to(dtype)


def _trained(gen, d_in, d_out, K, n_stored, dtype, clustered=False):
    """What training leaves: weight, mask, fan-in, bias."""
    return (_normal(gen, (d_out, d_in), K ** -0.5, dtype), _mask(gen, d_in, d_out, K, n_stored, clustered), K, _normal(gen, (d_out,), 0.1))


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    d_in, d_out, K, n = case["d_in"], case["d_out"], _fan_in(case), _stored(case)
    if case["kind"] == "forward":
        layer = condense_layer(*_trained(gen, d_in, d_out, K, n, _dtype(case), case["indices"] == "clustered"))
        if case["narrow"]:
            layer = layer.narrow()
        return {"kind": "forward", "layer": layer, "form": case["form"], "x": _normal(gen, (case["batch"], d_in), 1.0, _dtype(case))}
    if case["kind"] == "mlp":
        first = condense_layer(*_trained(gen, d_in, d_out, K, n, torch.float32))
        # the second layer's fan-in counts its stored inputs: what training with ablated hidden neurons leaves it
        second = condense_layer(*_trained(gen, d_out, d_in, _fan_in(case, n), d_in, torch.float32))
        return {"kind": "mlp", "block": fold_mlp(first, second, B_.ACT_GELU), "x": _normal(gen, (case["batch"], d_in), 1.0)}
    if case["kind"] == "condense":
        return {"kind": "condense", "trained": _trained(gen, d_in, d_out, K, n, _dtype(case))}
    W, mask, K, _ = _trained(gen, d_in, d_out, K, n, torch.float32)
    W *= mask
    return {"kind": "update", "W": W, "mask": mask, "grad": _normal(gen, (d_out, d_in), 1e-3), "K": K, "moved": n * K * case["moved"] // 100, "budget": n * K,
            "mask_out": torch.empty_like(mask), "W_out": torch.empty_like(W), "report": torch.empty((4,), dtype=torch.int64, device="cuda"),
            "workspace": torch.empty((B_.srigl_mask_update_workspace_bytes(d_out, d_in),), dtype=torch.uint8, device="cuda")}


def run(state):
    if state["kind"] == "forward":
        return state["layer"].forward(state["x"], representation=state["form"])
    if state["kind"] == "mlp":
        return state["block"].forward(state["x"])
    if state["kind"] == "condense":
        layer: CondensedLinear = condense_layer(*state["trained"])
        return {"W_c": layer.W_c, "idx": layer.idx, "active": layer.active, "seg": layer.seg, "packed": layer.packed, "n_active": layer.n_active}
    W, s = state["W"], state
    B_.srigl_mask_update(W, s["mask"], s["grad"], W.shape[0], W.shape[1], s["K"], s["moved"], 30, s["budget"], s["mask_out"], s["W_out"], s["workspace"],
                         s["report"])
    return s["mask_out"], s["W_out"], s["report"]


def work(case):
    """Each input read once and each output written once; 2 operations per stored weight and batch row."""
    d_in, d_out, K, n = case["d_in"], case["d_out"], _fan_in(case), _stored(case)
    size = 4 if case["dtype"] == "f32" else 2
    if case["kind"] == "forward":
        index = 2 if case["narrow"] else 4
        return {"bytes": n * K * (size + index) + case["batch"] * (d_in * size + d_out * 4) + 4 * (d_out + n), "flops": 2 * case["batch"] * n * K}
    if case["kind"] == "mlp":
        terms = n * K + d_in * _fan_in(case, n)
        return {"bytes": terms * 8 + case["batch"] * 8 * d_in + 4 * (d_in + 2 * n), "flops": 2 * case["batch"] * terms}
    if case["kind"] == "condense":
        packed = B_.srigl_packed_bytes(n, K, d_in, B_.F32 if size == 4 else B_.BF16)
        seg = n * B_.srigl_seg_stride(d_in) * 2
        # the mask whole; of the weights what the mask keeps
        return {"bytes": d_out * d_in + n * K * (2 * size + 4) + packed + seg + 4 * n, "flops": 0}
    return {"bytes": d_in * d_out * (4 + 4 + 1 + 4 + 1), "flops": 0}


def tolerance(case):
    # Condensing copies bits and an update ranks exact values.  The sums run in fp32 for both element types (products of
    # bf16 values are exact in fp32); only their order is free.
    return "exact" if case["kind"] in ("condense", "update") else {"rel": 1e-5}
