"""Workloads of the N:M-sparse linear library, as a program that uses it meets them.

Every workload goes through the public calls of the package.  Shapes are those of the transformer blocks in
`paper_2409_09708_amd.workloads` (four linears per block, images of 197 tokens, one N:M level per layer) and of
generic layers around them; values are the seeded Gaussians used throughout the repository (activations N(0, 1),
weights N(0, 0.02), int8 operands round(N(0, 40)) clipped to [-127, 127]).

A case is a dict of plain values; `kind` names what is done:
  layer    one linear layer.  call: "prepared" (weight in operand order once, the product on each call), "plain"
           (packed weight in, product out), "static" (the call that allocates nothing) or "packed" (no workspace: the
           product straight from the packed format)
  block    the four linears of one transformer block, one prepared call after another
  stages   one block per stage of a four-stage hierarchy (narrow and many tokens to wide and few), one call each
  stack    the independent products of a whole model in one batched call; compress: the weights are selected, packed
           and laid out for the products in the same pass
  train    one training step of a block: prune, pack, forward, input gradient and weight gradient of every linear
  int8     the four linears of a block on int8 operands
  nested   a supernet update: rank every weight once, pack the sampled configuration from the ranks
  scored   compression by a supplied saliency: mask from scores, pack under the mask, and back to the dense weight
"""
import math

import torch

import paper_2409_09708_amd as nm
from paper_2409_09708_amd import workloads as wl

INDEX_BITS = {4: 2, 8: 3, 16: 4}
LEVELS = list(wl.LEVELS_ALL)
TOKENS = 197  # per image
DTYPES = {"bf16": torch.bfloat16, "f32": torch.float32}


# ------------------------------------------------------------------------------------------------------
# cases
# ------------------------------------------------------------------------------------------------------
def listed():
    return [
        # the smallest call: one image through a narrow square projection of a deployed model; launch latency
        {"name": "layer_proj_1_image", "kind": "layer", "call": "prepared", "T": 197, "K": 384, "O": 384, "N": 2,
         "M": 4, "out": "bf16", "bias": False},
        # a classification head on a handful of tokens, called without any preparation
        {"name": "layer_head_8_tokens", "kind": "layer", "call": "plain", "T": 8, "K": 768, "O": 1000, "N": 4, "M": 8,
         "out": "f32", "bias": True},
        # an ordinary serving batch through the long reduction of the MLP
        {"name": "layer_fc2_8_images", "kind": "layer", "call": "prepared", "T": 1576, "K": 3072, "O": 768, "N": 1,
         "M": 16, "out": "bf16", "bias": True},
        # nothing fits a tile: odd token count, a width that is no multiple of 64, an odd number of out-features
        {"name": "layer_ragged", "kind": "layer", "call": "plain", "T": 1579, "K": 1000, "O": 1001, "N": 2, "M": 8,
         "out": "f32", "bias": True},
        # one image through every linear of a 12-block model (independent products): latency, weights from HBM
        {"name": "stack_1_image", "kind": "stack", "C": 768, "blocks": 12, "batch": 1, "level_seed": 0,
         "compress": False},
        # compression and products of the whole model at a throughput batch: the largest case
        {"name": "stack_256_images", "kind": "stack", "C": 768, "blocks": 12, "batch": 256, "level_seed": 0,
         "compress": True},
        # a deployed block at a serving batch, its layers one after another as a model runs them
        {"name": "block_64_images", "kind": "block", "C": 768, "batch": 64, "level_seed": 0, "out": "bf16",
         "bias": True},
        # the same for a hierarchy: 16 layers from 200704 tokens x 128 to 3136 tokens x 1024
        {"name": "stages_64_images", "kind": "stages", "batch": 64, "level_seed": 0},
        # a training step of one block: both directions, weights changing from step to step
        {"name": "train_block_64_images", "kind": "train", "C": 768, "batch": 64, "N": 2, "M": 8, "grad": "f32",
         "masked": True},
        # the quantised block at a serving batch, weights kept in their compressed form
        {"name": "int8_block_64_images", "kind": "int8", "C": 768, "batch": 64, "level_seed": 0, "form": "packed",
         "out": "bf16"},
        # supernet training: all 48 weights of a 12-block model ranked, one configuration packed
        {"name": "nested_12_blocks", "kind": "nested", "C": 768, "blocks": 12, "M": 8, "level_seed": 0},
        # one block compressed by an external (Taylor) score and expanded again
        {"name": "scored_block", "kind": "scored", "C": 768, "N": 2, "M": 4},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _width(rng):
    """A model width: the ones of the repository's workloads, or a generic multiple of 32."""
    return rng.choice([128, 256, 384, 512, 768, 1024, 32 * rng.randint(4, 32)])


def draw(rng):
    kind = rng.choice(["layer", "layer", "layer", "layer", "block", "stack", "train", "int8", "nested", "scored"])
    N, M = rng.choice(LEVELS)
    if kind == "layer":
        call = rng.choice(["prepared", "prepared", "plain", "static", "packed"])
        T, K, O = _log_int(rng, 1, 50432), _log_int(rng, 64, 4096), _log_int(rng, 64, 4096)
        K = max(M, K // M * M) if rng.random() < 0.25 else max(64, K // 64 * 64)
        if rng.random() < 0.75:
            O = max(64, O // 8 * 8)
        if call == "static":  # the operand-order copy has to fit the library's fixed scratch
            K, O = min(K, 1024), min(O, 2048)
        if call == "packed":  # what the packed-format path takes
            T, K, O = min(T, _log_int(rng, 1, 208)), max(64, K // 64 * 64), O // 4 * 4
            N, M = rng.choice(wl.LEVELS_7)
        if T * K * O > 50432 * 768 * 3072:
            T = 50432 * 768 * 3072 // (K * O)
        if (K % 64 or O % 8) and T * K * O > 4096 * 1024 * 1024:
            T = max(1, 4096 * 1024 * 1024 // (K * O))
        return {"kind": kind, "call": call, "T": T, "K": K, "O": O, "N": N, "M": M,
                "out": rng.choice(["bf16", "f32"]), "bias": rng.random() < 0.5}
    C, seed = _width(rng), rng.randint(0, 1 << 20)
    if kind == "block":
        return {"kind": kind, "C": C, "batch": _log_int(rng, 1, 256), "level_seed": seed,
                "out": rng.choice(["bf16", "bf16", "f32"]), "bias": rng.random() < 0.5}
    if kind == "stack":
        blocks = rng.randint(1, 12)
        return {"kind": kind, "C": min(C, 768), "blocks": blocks, "batch": _log_int(rng, 1, 256), "level_seed": seed,
                "compress": rng.random() < 0.5}
    if kind == "train":
        return {"kind": kind, "C": C, "batch": _log_int(rng, 1, 128), "N": N, "M": M,
                "grad": rng.choice(["f32", "bf16"]), "masked": rng.random() < 0.75}
    if kind == "int8":
        return {"kind": kind, "C": max(128, C // 128 * 128), "batch": _log_int(rng, 1, 256), "level_seed": seed,
                "form": rng.choice(["packed", "dense"]), "out": rng.choice(["bf16", "f32", "i32"])}
    if kind == "nested":
        return {"kind": kind, "C": C, "blocks": rng.randint(1, 12), "M": M, "level_seed": seed}
    return {"kind": kind, "C": C, "N": N, "M": M}


# ------------------------------------------------------------------------------------------------------
# inputs
# ------------------------------------------------------------------------------------------------------
class _Draws:
    """Seeded device-side draws."""

    def __init__(self, seed):
        self.gen = torch.Generator(device="cuda")
        self.gen.manual_seed(int(seed))

    def normal(self, *shape, std=1.0, dtype=torch.bfloat16):
        return torch.empty(*shape, dtype=dtype, device="cuda").normal_(0.0, std, generator=self.gen)

    def weight(self, O, K):
        return self.normal(O, K, std=0.02)

    def int8(self, rows, cols):
        return self.normal(rows, cols, std=40.0, dtype=torch.float32).round_().clamp_(-127, 127).to(torch.int8)


def _levels(case, count):
    return wl.draw_levels(case["level_seed"], wl.LEVELS_7, count)


def _block_layers(case):
    """The linears of a case as wl.Layer records."""
    kind = case["kind"]
    if kind == "layer":
        return [wl.Layer("layer", case["T"], case["K"], case["O"], case["N"], case["M"])]
    if kind == "stages":
        return wl.swin_b_stages(case["batch"], case["level_seed"])
    blocks, T = case.get("blocks", 1), case.get("batch", 1) * TOKENS
    if kind in ("train", "scored"):
        levels = [(case["N"], case["M"])] * 4
    elif kind == "nested":
        levels = wl.draw_levels(case["level_seed"], [lv for lv in wl.LEVELS_7 if lv[1] == case["M"]], 4 * blocks)
    else:
        levels = _levels(case, 4 * blocks)
    return [wl.Layer(f"{b}.{name}", T, K, O, *levels[4 * b + i])
            for b in range(blocks) for i, (name, K, O) in enumerate(wl.block_shapes(case["C"]))]


def _flat_views(sizes, dtype):
    """One buffer and its consecutive pieces (256-byte aligned) of the given 2-D sizes."""
    step = 256 // torch.empty(0, dtype=dtype).element_size()
    starts, end = [], 0
    for r, c in sizes:
        starts.append(end)
        end += -(-r * c // step) * step
    buf = torch.zeros(end, dtype=dtype, device="cuda")
    return buf, [buf[s:s + r * c].view(r, c) for s, (r, c) in zip(starts, sizes)]


def prepare(case, seed):
    d, kind = _Draws(seed), case["kind"]
    layers = _block_layers(case)
    state = {"case": dict(case), "layers": layers}
    if kind in ("layer", "block", "stages"):
        items = []
        for L in layers:
            W, X = d.weight(L.O, L.K), d.normal(L.T, L.K)
            values, indices = nm.nm_pack(W, L.N, L.M)
            bias = d.normal(L.O, std=0.1, dtype=torch.float32) if case.get("bias") else None
            out = torch.zeros(L.T, L.O, dtype=DTYPES[case.get("out", "bf16")], device="cuda")
            ws = None
            if case.get("call", "prepared") == "prepared":
                ws = nm.nm_spmm_prepare(values, indices, L.K, L.N, L.M, L.T)
            items.append((values, indices, X, ws, bias, out))
        state["items"] = items
    elif kind == "stack":
        Ws = [d.weight(L.O, L.K) for L in layers]
        Xs = [d.normal(L.T, L.K) for L in layers]
        state["values"], values = _flat_views([(L.O, L.K // L.M * L.N) for L in layers], torch.bfloat16)
        state["indices"], indices = _flat_views(
            [(L.O, nm.nm_index_bytes(L.O, L.K, L.N, L.M) // (4 * L.O)) for L in layers], torch.int32)
        state["outputs"], ys = [], []
        for b in range(0, len(layers), 4):
            buf, views = _flat_views([(L.T, L.O) for L in layers[b:b + 4]], torch.bfloat16)
            state["outputs"].append(buf)
            ys += views
        state["pack"] = [(W, L.N, L.M, L.T) for W, L in zip(Ws, layers)]
        state["packed"] = list(zip(values, indices))
        _, state["workspaces"] = nm.nm_pack_prepare_batched(state["pack"], out=state["packed"])
        state["descs"] = nm.forward_descs(
            [(v, i, L.K, L.N, L.M, X, ws, None, y)
             for L, v, i, X, ws, y in zip(layers, values, indices, Xs, state["workspaces"], ys)])
        state["keep"] = (Xs, ys)
    elif kind == "train":
        state["items"] = []
        for L in layers:
            W, X, dY = d.weight(L.O, L.K), d.normal(L.T, L.K), d.normal(L.T, L.O)
            state["items"].append((W, torch.empty_like(W), X, dY))
    elif kind == "int8":
        state["items"] = []
        for L in layers:
            Wq, Xq = d.int8(L.O, L.K), d.int8(L.T, L.K)
            mask = nm.nm_prune(Wq.to(torch.bfloat16), L.N, L.M)
            w_scale = d.normal(L.O, std=0.1, dtype=torch.float32).exp_().mul_(0.0005)
            bias = d.normal(L.O, std=0.1, dtype=torch.float32)
            if case["form"] == "packed":
                weight = nm.nm_pack_i8(Wq, mask, L.N, L.M)
                ws = nm.nm_i8_prepare_packed(*weight, L.K, L.N, L.M, L.T)
            else:
                weight = (Wq, mask)
                ws = nm.nm_i8_prepare(Wq, mask, L.N, L.M, L.T)
            dtype = torch.int32 if case["out"] == "i32" else DTYPES[case["out"]]
            state["items"].append((weight, Xq, ws, w_scale, bias, torch.zeros(L.T, L.O, dtype=dtype, device="cuda")))
    elif kind == "nested":
        Ws = [d.weight(L.O, L.K) for L in layers]
        state["ranks"], ranks = _flat_views([(L.O, L.K // 2) for L in layers], torch.uint8)
        state["values"], values = _flat_views([(L.O, L.K // L.M * L.N) for L in layers], torch.bfloat16)
        state["indices"], indices = _flat_views(
            [(L.O, nm.nm_index_bytes(L.O, L.K, L.N, L.M) // (4 * L.O)) for L in layers], torch.int32)
        state["rank"] = [(W, L.M) for W, L in zip(Ws, layers)]
        state["rank_out"] = ranks
        state["pack"] = [(W, r, L.N, L.M) for W, r, L in zip(Ws, ranks, layers)]
        state["packed"] = list(zip(values, indices))
    else:
        state["items"] = []
        for L in layers:
            W = d.weight(L.O, L.K)
            score = W.float().mul_(d.normal(L.O, L.K, dtype=torch.float32)).abs_()  # |weight * gradient|
            state["items"].append((W, score))
    return state


# ------------------------------------------------------------------------------------------------------
# one pass
# ------------------------------------------------------------------------------------------------------
def run(state):
    case, layers = state["case"], state["layers"]
    kind = case["kind"]
    if kind in ("layer", "block", "stages"):
        outs, call = [], case.get("call", "prepared")
        for L, (values, indices, X, ws, bias, out) in zip(layers, state["items"]):
            if call == "prepared":
                nm.nm_linear_forward_prepared(values, indices, L.K, L.N, L.M, X, ws, bias=bias, out=out)
            elif call == "static":
                nm.nm_linear_forward_static(values, indices, L.K, L.N, L.M, X, bias=bias, out=out)
            else:
                nm.nm_linear_forward(values, indices, L.K, L.N, L.M, X, bias=bias, out=out,
                                     from_packed=call == "packed")
            outs.append(out)
        return outs
    if kind == "stack":
        if case["compress"]:
            nm.nm_pack_prepare_batched(state["pack"], out=state["packed"], workspaces=state["workspaces"])
        nm.nm_linear_forward_prepared_batched(state["descs"])
        packed = [state["values"].view(torch.int16), state["indices"]] if case["compress"] else []
        return state["outputs"] + packed
    if kind == "train":
        outs, grad = [], DTYPES[case["grad"]]
        for L, (W, Wm, X, dY) in zip(layers, state["items"]):
            mask = nm.nm_prune(W, L.N, L.M, W_masked=Wm)
            values, indices = nm.nm_pack(W, L.N, L.M, mask=mask)
            Y = nm.nm_linear_forward(values, indices, L.K, L.N, L.M, X, out_dtype=torch.bfloat16)
            dX = nm.nm_linear_backward_input(Wm, dY, out_dtype=torch.bfloat16)
            dW = nm.nm_linear_backward_weight(dY, X, mask=mask if case["masked"] else None, out_dtype=grad)
            outs += [mask, Y, dX, dW]
        return outs
    if kind == "int8":
        outs = []
        for L, (weight, Xq, ws, w_scale, bias, out) in zip(layers, state["items"]):
            if case["form"] == "packed":
                nm.nm_linear_forward_i8_packed_prepared(*weight, L.K, L.N, L.M, Xq, ws, x_scale=0.02, w_scale=w_scale,
                                                        bias=bias, out=out)
            else:
                nm.nm_linear_forward_i8_prepared(*weight, L.N, L.M, Xq, ws, x_scale=0.02, w_scale=w_scale, bias=bias,
                                                 out=out)
            outs.append(out)
        return outs
    if kind == "nested":
        nm.nm_rank_batched(state["rank"], out=state["rank_out"])
        nm.nm_pack_ranked_batched(state["pack"], out=state["packed"])
        return [state["ranks"], state["values"].view(torch.int16), state["indices"]]
    outs = []
    for L, (W, score) in zip(layers, state["items"]):
        mask = nm.nm_prune_scored(score, L.N, L.M)
        values, indices = nm.nm_pack(W, L.N, L.M, mask=mask)
        dense = nm.nm_unpack(values, indices, L.K, L.N, L.M)
        outs += [mask, values.view(torch.int16), indices, dense.view(torch.int16)]
    return outs


# ------------------------------------------------------------------------------------------------------
# what a pass cannot do without, and how far two correct results may lie apart
# ------------------------------------------------------------------------------------------------------
def _packed_bytes(L, value_bytes=2):
    fields = L.K // L.M * L.N
    return L.O * (fields * value_bytes + (fields * INDEX_BITS[L.M] + 31) // 32 * 4)


def _mask_bytes(L):
    return L.O * ((L.K + 31) // 32) * 4


def work(case):
    kind = case["kind"]
    out = {"bf16": 2, "f32": 4, "i32": 4}[case.get("out", "bf16")]
    nbytes = flops = 0
    for L in _block_layers(case):
        if kind in ("layer", "block", "stages", "stack"):
            nbytes += 2 * L.T * L.K + _packed_bytes(L) + out * L.T * L.O + (4 * L.O if case.get("bias") else 0)
            nbytes += 2 * L.O * L.K if case.get("compress") else 0
            flops += L.useful_flops
        elif kind == "train":
            grad = 4 if case["grad"] == "f32" else 2
            nbytes += 2 * L.O * L.K + _mask_bytes(L) + 2 * L.T * L.K + 2 * L.T * L.O  # W, mask, X, dY
            nbytes += 2 * L.T * L.O + 2 * L.T * L.K + grad * L.O * L.K                # Y, dX, dW
            flops += L.useful_flops + 2 * L.dense_flops
        elif kind == "int8":
            weight = _packed_bytes(L, 1) if case["form"] == "packed" else L.O * L.K + _mask_bytes(L)
            nbytes += L.T * L.K + weight + out * L.T * L.O + 8 * L.O
            flops += L.useful_flops
        elif kind == "nested":
            nbytes += 2 * L.O * L.K + L.O * L.K // 2 + _packed_bytes(L)
        else:
            nbytes += (4 + 2 + 2) * L.O * L.K + _mask_bytes(L) + _packed_bytes(L)
    return {"bytes": float(nbytes), "flops": float(flops)}


def tolerance(case):
    """Compression and int8 sums are exact by definition.  Products of bfloat16 operands are exact in fp32, so two
    correct results differ by the order of an fp32 sum (measured against fp64 sums on the listed shapes: 2-norm 3e-7,
    largest 2e-6 of the rms) and, for bfloat16 outputs, by its rounding (2-norm 1.7e-3, largest 3.9e-3 of the
    value).  Four times what is measured is stated."""
    kind = case["kind"]
    if kind in ("nested", "scored", "int8"):
        return "exact"
    f32_only = case.get("out") == "f32" and kind != "train"
    return {"rel": 1.2e-6, "max": 8e-6} if f32_only else {"rel": 6.6e-3, "max": 1.6e-2}
