"""What the speed of this library is judged by: bags of packed variable-length sequences, from the
smallest call to the largest benchmark bag, through the public Python entry points.

A case is a plain dict.  ``kind`` says which calls one pass makes:

* ``train``    forward and backward of one bag (one attention layer of a training step); ``causal``
               selects the causal pair of entry points;
* ``forward``  the forward alone (sampling, or the frozen half of a distillation step);
* ``ulysses``  what one GPU of a ``g``-GPU bag does to its own data around the two all-to-alls of one
               attention call: heads of q, k, v packed for sending, the received chunks of q, k, v put
               together, the attention output cut back into chunks, the returned heads unpacked; with
               ``plan`` the bag is new and its row map is built in the same pass.

``lens`` lists the sequence lengths of the bag in packing order (text, comma separated), ``H`` and ``d``
the heads and the head dimension (for ``ulysses``: before the switch).
"""
from __future__ import annotations

import math
import random
from typing import Dict, List

import torch

import paper_2508_06001_amd as K

# text + image tokens at 24 heads of 128, the mixed-resolution benchmark bag (31464 tokens)
MIXED_RES = "1406,4130,361,328,4079,2615,1407,1355,502,1306,4533,2686,367,1413,1141,1359,2476"
# images and video clips, the image+video benchmark bag (66792 tokens)
IMAGE_VIDEO = "1401,2617,7955,4124,8033,14415,559,8302,1064,484,1211,7977,406,8244"
# one GPU's post-switch share of an 8-GPU bag (3 of 24 heads)
POST_ULYSSES = "131072,32768,8192,8192,8192,8192"

IMAGE_TOKENS = (256, 1024, 2304, 4096, 4032)
VIDEO_TOKENS = (5 * 1560, 9 * 1560, 16 * 1560)
# heads x head dimension: the 24-head model whole and as 2-, 4- and 8-GPU shares, and the d = 64 families
SHAPES = ((24, 128), (24, 128), (24, 128), (12, 128), (6, 128), (3, 128), (48, 64), (12, 64), (2, 64))
MOST_FLOPS = 1.8e14          # of a drawn case: below the largest listed one
MOST_TOKENS = 131072


def _text(lens) -> str:
    return ",".join(str(int(x)) for x in lens)


def _low_res() -> str:
    """One GPU's share of the paper's low-resolution stream: 32 images of 256 tokens, 0 to 392 text tokens each."""
    rng = random.Random(256)
    return _text(256 + rng.randint(0, 392) for _ in range(32))


def _skewed() -> str:
    """One long sequence and 200 short ones."""
    rng = random.Random(65536)
    return _text([65536] + [rng.randint(200, 400) for _ in range(200)])


def listed() -> List[Dict]:
    return [
        # the smallest call: four short sequences of two 64-wide heads, where launches and latency are all there is
        {"name": "tiny", "kind": "train", "lens": "37,128,200,311", "H": 2, "d": 64, "causal": False},
        # sampling one 1024 x 1024 image, conditional and unconditional prompt in one bag: forward only
        {"name": "sample_image_pair", "kind": "forward", "lens": "4173,4096", "H": 24, "d": 128, "causal": False},
        # one GPU's share of the low-resolution stream: short, ragged sequences
        {"name": "low_res", "kind": "train", "lens": _low_res(), "H": 24, "d": 128, "causal": False},
        # a balanced bag that is one 1024 x 1024 image and its caption: too few tiles to fill the GPU evenly
        {"name": "single_image", "kind": "train", "lens": "4292", "H": 24, "d": 128, "causal": False},
        # the mixed-resolution training bag
        {"name": "mixed_res", "kind": "train", "lens": MIXED_RES, "H": 24, "d": 128, "causal": False},
        # the same bag under the causal mask
        {"name": "mixed_res_causal", "kind": "train", "lens": MIXED_RES, "H": 24, "d": 128, "causal": True},
        # the joint stream at 48 heads of 64: clips of 25 low-resolution frames, images and short sequences
        {"name": "joint_d64", "kind": "train", "lens": "6513,6795,4344,1221,1268,433,310,589,452,351", "H": 48, "d": 64,
         "causal": False},
        # images and videos
        {"name": "image_video", "kind": "train", "lens": IMAGE_VIDEO, "H": 24, "d": 128, "causal": False},
        # the headline bag, and the largest: one 65536-token sequence among 200 short ones, peaky keys
        {"name": "skewed", "kind": "train", "lens": _skewed(), "H": 24, "d": 128, "causal": False, "peaky": True},
        # one GPU's share of a sequence-parallel bag: three heads, very long sequences
        {"name": "post_ulysses", "kind": "train", "lens": POST_ULYSSES, "H": 3, "d": 128, "causal": False},
        # a new two-GPU bag of one batch: the row map and one layer's data movement
        {"name": "switch_small", "kind": "ulysses", "lens": "1024,1391,4096,4211,613", "H": 24, "d": 128, "g": 2, "plan": True},
        # one layer's data movement of the 8-GPU bag behind post_ulysses
        {"name": "switch_large", "kind": "ulysses", "lens": POST_ULYSSES, "H": 24, "d": 128, "g": 8, "plan": False},
    ]


def _lens(case: Dict) -> List[int]:
    return [int(x) for x in case["lens"].split(",")]


def _pairs(case: Dict) -> float:
    """Query-key pairs the mask leaves, over all sequences, per head."""
    if case["causal"]:
        return sum(l * (l + 1) / 2.0 for l in _lens(case))
    return sum(float(l) * l for l in _lens(case))


def _flops(case: Dict) -> float:
    if case["kind"] == "ulysses":
        return 0.0
    return (14.0 if case["kind"] == "train" else 4.0) * case["H"] * case["d"] * _pairs(case)


def _log_int(rng: random.Random, lo: int, hi: int) -> int:
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_lens(rng: random.Random) -> List[int]:
    """A bag of one of the families above, its tokens spread over the logarithm of the range."""
    tokens = _log_int(rng, 600, MOST_TOKENS)
    family = rng.choice(("images", "images", "image_video", "low_res", "single", "equal", "skewed"))
    if family == "single":
        return [tokens]
    if family == "skewed":
        return [max(1, tokens // 2)] + [rng.randint(200, 400) for _ in range(max(1, tokens // 600))]
    if family == "equal":
        n = _log_int(rng, 1, min(256, max(1, tokens // 64)))
        return [tokens // n] * n
    lens: List[int] = []
    while sum(lens) < tokens:
        if family == "low_res":
            new = 256 + rng.randint(0, 392)
        elif family == "image_video" and rng.random() < 0.5:
            new = rng.choice(VIDEO_TOKENS) + rng.randint(64, 512)
        else:
            new = rng.choice(IMAGE_TOKENS) + rng.randint(16, 512)
        left = tokens - sum(lens)
        lens.append(new if new <= left or left < 300 else rng.randint(left // 2, left))
    return lens


def draw(rng: random.Random) -> Dict:
    kind = rng.choice(("train", "train", "train", "train", "forward", "ulysses"))
    if kind == "ulysses":
        g = rng.choice((2, 4, 8))
        return {"kind": kind, "lens": _text(_draw_lens(rng)), "H": 24, "d": 128, "g": g, "plan": rng.random() < 0.5}
    while True:
        H, d = rng.choice(SHAPES)
        case = {"kind": kind, "lens": _text(_draw_lens(rng)), "H": H, "d": d, "causal": rng.random() < 0.25}
        if kind == "train" and rng.random() < 0.15:
            case["peaky"] = True
        if _flops(case) <= MOST_FLOPS:
            return case


def _normal(gen: torch.Generator, shape) -> torch.Tensor:
    return torch.randn(shape, generator=gen, dtype=torch.bfloat16, device="cuda")


def prepare(case: Dict, seed: int) -> Dict:
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    lens, H, d = _lens(case), case["H"], case["d"]
    T = sum(lens)
    cu = [0]
    for l in lens:
        cu.append(cu[-1] + l)
    if case["kind"] == "ulysses":
        g = case["g"]
        n = len(lens)
        t_local = K.knap_ulysses_local_tokens(lens, g)[0]
        full, local = (T, H // g, d), (t_local, H, d)
        state = {
            "case": case, "n": n, "T": T, "t_local": t_local,
            "cu": torch.tensor(cu, dtype=torch.int32, device="cuda"),
            "row_map": torch.empty((T,), dtype=torch.int32, device="cuda"),
            "workspace": torch.empty((max(256, K.knap_ulysses_plan_workspace_bytes(n, g)),), dtype=torch.uint8, device="cuda"),
            # this GPU's q, k, v; what arrived for it; the attention's output; what came back
            "qkv": [_normal(gen, local) for _ in range(3)],
            "recv": [_normal(gen, full) for _ in range(3)],
            "out": _normal(gen, full),
            "back": _normal(gen, local),
            "packed": [torch.empty(local, dtype=torch.bfloat16, device="cuda") for _ in range(3)],
            "whole": [torch.empty(full, dtype=torch.bfloat16, device="cuda") for _ in range(3)],
            "send": torch.empty(full, dtype=torch.bfloat16, device="cuda"),
            "x": torch.empty(local, dtype=torch.bfloat16, device="cuda"),
        }
        if not case["plan"]:     # the bag's row map serves every layer: made once, before the pass
            K.knap_ulysses_plan(state["cu"], n, T, g, state["row_map"], state["workspace"])
        return state
    attn = K.VarlenAttention(cu, H, d, 1.0 / math.sqrt(d), causal=case["causal"])
    q, k, v = (_normal(gen, (T, H, d)) for _ in range(3))
    if case.get("peaky"):        # one key entry in a hundred is eight times as large
        for r in range(0, T, 16384):
            rows = k[r:r + 16384]
            rows.mul_(1 + 7 * (torch.rand(rows.shape, generator=gen, device="cuda") < 0.01).to(torch.bfloat16))
    dout = _normal(gen, (T, H, d)) if case["kind"] == "train" else None
    return {"case": case, "attn": attn, "q": q, "k": k, "v": v, "dout": dout}


def run(state: Dict):
    case = state["case"]
    if case["kind"] == "ulysses":
        H, d, g = case["H"], case["d"], case["g"]
        T, t_local, hg = state["T"], state["t_local"], case["H"] // case["g"]
        if case["plan"]:
            K.knap_ulysses_plan(state["cu"], state["n"], T, g, state["row_map"], state["workspace"])
        for x, y in zip(state["qkv"], state["packed"]):
            K.knap_ulysses_pack_heads(x, t_local, H, d, g, y)
        for x, y in zip(state["recv"], state["whole"]):
            K.knap_ulysses_gather_chunks(x, state["row_map"], T, hg, d, y)
        K.knap_ulysses_scatter_chunks(state["out"], state["row_map"], T, hg, d, state["send"])
        K.knap_ulysses_unpack_heads(state["back"], t_local, H, d, g, state["x"])
        return {"row_map": state["row_map"], "packed": state["packed"], "whole": state["whole"], "send": state["send"],
                "x": state["x"]}
    attn = state["attn"]
    out, lse = attn.forward(state["q"], state["k"], state["v"])
    if case["kind"] == "forward":
        return {"out": out, "lse": lse}
    dq, dk, dv = attn.backward(state["q"], state["k"], state["v"], state["dout"])
    return {"out": out, "lse": lse, "dq": dq, "dk": dk, "dv": dv}


def work(case: Dict) -> Dict:
    lens, H, d = _lens(case), case["H"], case["d"]
    T = sum(lens)
    if case["kind"] == "ulysses":
        g = case["g"]
        t_local = sum(l // g + (1 if l % g else 0) for l in lens)     # chunk 0 of every sequence
        moved = 4 * t_local * H * d * 2 + 4 * T * (H // g) * d * 2    # four tensors of each layout
        return {"bytes": 2 * moved + 4 * T, "flops": 0}
    tensor = 2 * T * H * d
    n = 8 if case["kind"] == "train" else 4      # q, k, v, dout in; out, dq, dk, dv out
    return {"bytes": n * tensor + 4 * T * H, "flops": _flops(case)}


def tolerance(case: Dict):
    if case["kind"] == "ulysses":
        return "exact"
    # About four times the distance of the present outputs from the same path in float64 (worst of out, lse, dq,
    # dk, dv): rel 2.9e-3 on every bag (the bf16 rounding of the stored result); max 0.03 on the bidirectional
    # bags, 0.10 under the causal mask (its first rows see one or two keys), 0.48 with peaky keys (a near one-hot
    # row's dq is a small difference of large terms).
    if case.get("peaky"):
        return {"rel": 1e-2, "max": 0.95}
    return {"rel": 1e-2, "max": 0.4 if case["causal"] else 0.12}
