"""The work that users of this package have it do, as timed cases.

Five kinds of work, each through the package's public entry points:

``step``      one pack -> attention -> unpack layer as ONE launch (binding.ragged_pack_attn_unpack), the call of a
              serving loop; ``eager`` calls the checked binding, otherwise the pre-marshalled call is re-issued.
``stages``    the same layer as its three separate calls, which is what a program uses that puts work of its own
              between the stages.
``attn``      ragged attention in place on a fused [T, 3, H, D] QKV buffer, between two linear layers.
``padded``    one attention layer on the padded layout (binding.ragged_attn_padded).
``prune``     the pruning decision and the data movement around it: scores, top-k mask, pack, zero-filling unpack.
``blocks``    encoder blocks on packed rows behind a given keep mask (harness.PackedBlocks), captured in a graph.
``encoder``   a whole encoder that prunes on its way (harness.ProgressiveBlocks), captured in a graph.

Geometry is that of the DeiT encoders the package's workloads name: head dim 64, 3 / 6 / 12 heads, 197 tokens at
224 x 224 and 577 at 384 x 384, plus generic odd sizes in the drawn cases.  Inputs are N(0, 1) features and
seeded Bernoulli keep masks that always keep the class token.
"""
import math

import torch

from paper_2604_15408_amd import binding, harness
from paper_2604_15408_amd import workloads as wl

DEV = "cuda:0"
D = 64
_DTYPES = {"f16": torch.float16, "bf16": torch.bfloat16, "f32": torch.float32}


def listed():
    return [
        # the smallest call: two images of a 3-head model, one layer, through the checked eager binding
        {"name": "step_tiny_eager", "kind": "step", "B": 2, "N": 197, "H": 3, "keep": 0.6, "dtype": "f16", "fill": 0, "eager": True},
        # interactive serving of two 384 x 384 images: latency of a single pre-marshalled launch
        {"name": "step_384_bs2", "kind": "step", "B": 2, "N": 577, "H": 12, "keep": 0.3, "dtype": "f16", "fill": 0, "eager": False},
        # the ordinary serving batch: DeiT-B at 80 % pruned
        {"name": "step_bs32_keep20", "kind": "step", "B": 32, "N": 197, "H": 12, "keep": 0.2, "dtype": "f16", "fill": 0, "eager": False},
        # lightly pruned bf16 batch, three calls, every output byte defined
        {"name": "stages_bs64_bf16", "kind": "stages", "B": 64, "N": 197, "H": 12, "keep": 0.8, "dtype": "bf16", "fill": 1, "eager": False},
        # attention of an unpruned 384 x 384 layer in front of the pruning point, fused QKV, bf16
        {"name": "attn_384_bf16", "kind": "attn", "B": 32, "N": 577, "H": 12, "keep": 1.0, "dtype": "bf16", "out": "bf16"},
        # a pruned 384 x 384 batch that stays in the padded layout, zero fill
        {"name": "padded_384_bs32", "kind": "padded", "B": 32, "N": 577, "H": 12, "keep": 0.3, "dtype": "f16", "out": "f16", "fill": 1},
        # mask producer and packing of a large throughput batch
        {"name": "prune_bs256", "kind": "prune", "B": 256, "N": 197, "H": 12, "keep": 0.5, "dtype": "f16"},
        # eight late blocks of a small batch at half the tokens
        {"name": "blocks_bs8_keep50", "kind": "blocks", "B": 8, "N": 197, "H": 12, "keep": 0.5, "dtype": "f16", "depth": 8, "hint": True},
        # eight late blocks of the ordinary serving batch
        {"name": "blocks_bs32_keep20", "kind": "blocks", "B": 32, "N": 197, "H": 12, "keep": 0.2, "dtype": "f16", "depth": 8, "hint": True},
        # late blocks in bf16 on a large, lightly pruned batch, nothing known about the row count on the host
        {"name": "blocks_bs64_bf16", "kind": "blocks", "B": 64, "N": 197, "H": 12, "keep": 0.7, "dtype": "bf16", "depth": 8, "hint": False},
        # a DeiT-S sized encoder that prunes progressively in front of blocks 3, 6 and 9
        {"name": "encoder_small_bs32", "kind": "encoder", "B": 32, "N": 197, "H": 6, "keep": 0.7, "dtype": "f16", "depth": 12, "prune_at": "3,6,9"},
        # the throughput job: DeiT-B encoder, 128 images, pruned once to half
        {"name": "encoder_base_bs128", "kind": "encoder", "B": 128, "N": 197, "H": 12, "keep": 0.5, "dtype": "f16", "depth": 12, "prune_at": "4"},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same ranges: any batch up to the listed largest, odd token counts, 3 to 16 heads."""
    kind = rng.choice(("step", "step", "stages", "attn", "padded", "prune", "blocks", "blocks", "encoder"))
    case = {"kind": kind, "B": _log_int(rng, 1, 128), "N": rng.choice((197, 577, _log_int(rng, 40, 900))),
            "H": rng.choice((3, 6, 12, 12, 16)), "keep": round(rng.uniform(0.1, 1.0), 2), "dtype": rng.choice(("f16", "bf16"))}
    if kind in ("blocks", "encoder"):
        # transformer blocks cost most: at most as many rows as the largest listed case has, at most its width
        case["N"] = rng.choice((197, 197, _log_int(rng, 65, 577)))
        case["H"] = rng.choice((3, 6, 12))
        case["B"] = _log_int(rng, 1, max(2, min(128, 64 * 197 // case["N"])))
        case["depth"] = rng.choice((4, 8, 12))
    if kind == "step":
        case.update(fill=rng.choice((0, 1)), eager=rng.choice((False, False, True)))
    elif kind == "stages":
        case.update(fill=rng.choice((0, 1)), eager=False)
    elif kind == "attn":
        case.update(out=rng.choice((case["dtype"], "f32")))
    elif kind == "padded":
        case.update(out=rng.choice((case["dtype"], "f32")), fill=rng.choice((0, 1)))
    elif kind == "prune":
        case["B"] = _log_int(rng, 1, 256)
        case["N"] = rng.choice((197, 577, _log_int(rng, 40, 577)))
        case["keep"] = min(case["keep"], 0.9)
        if case["B"] * case["N"] * case["H"] > 256 * 197 * 12:
            case["B"] = max(1, 256 * 197 * 12 // (case["N"] * case["H"]))
    elif kind == "blocks":
        case.update(hint=rng.choice((True, False)))
    elif kind == "encoder":
        case["dtype"] = "f16"
        case["keep"] = rng.choice((0.5, 0.7))
        case["prune_at"] = {4: "2", 8: "3,6", 12: rng.choice(("4", "3,6,9"))}[case["depth"]]
    return case


def _prune_at(case):
    return tuple(int(s) for s in case["prune_at"].split(","))


def _kept(case):
    """Tokens kept per image by the top-k mask."""
    return max(1, int(round(case["keep"] * case["N"])))


def _randn(gen, dtype, *shape):
    return torch.randn(*shape, generator=gen, device=DEV, dtype=torch.float32).to(_DTYPES[dtype])


def prepare(case, seed):
    kind, B, N, H = case["kind"], case["B"], case["N"], case["H"]
    C, dt = H * D, _DTYPES[case["dtype"]]
    zeros = lambda *shape, dtype=dt: torch.zeros(*shape, dtype=dtype, device=DEV)
    if kind == "encoder":
        enc = harness.ProgressiveBlocks(B=B, N=N, H=H, D=D, depth=case["depth"], prune_at=_prune_at(case),
                                        keep_ratio=case["keep"], dtype=case["dtype"], seed=10 * int(seed) + 3000)
        return {"kind": kind, "obj": enc, "graph": harness.capture(torch, enc.run)}
    gen = torch.Generator(device=DEV).manual_seed(int(seed) * 7919 + 1)
    if kind == "prune":
        return {"kind": kind, "k": _kept(case), "x": _randn(gen, case["dtype"], B, N, C),
                "scores": zeros(B, N, dtype=torch.float64), "keep": zeros(B, N, dtype=torch.uint8),
                "packed": zeros(B * N, C), "cu": zeros(B + 1, dtype=torch.int32),
                "gidx": zeros(B * N, dtype=torch.int32), "out": zeros(B, N, C)}
    keep = wl.keep_bernoulli(B, N, case["keep"], int(seed) * 31 + 7)
    if kind == "blocks":
        w = wl.Workload("blocks", B, N, H, D, case["dtype"], int(seed) + 1, keep)
        hint = int(round(B * (1 + (N - 1) * case["keep"]))) if case["hint"] else 0
        pb = harness.PackedBlocks(w, case["depth"], rows_hint=hint)
        return {"kind": kind, "obj": pb, "graph": harness.capture(torch, pb.run)}
    kept = int(keep.sum())
    keep = keep.to(DEV)
    scale = D ** -0.5
    if kind == "attn":
        qkv = _randn(gen, case["dtype"], kept, 3, H, D)
        cu = torch.zeros(B + 1, dtype=torch.int32)
        cu[1:] = torch.cumsum(keep.cpu().to(torch.int32).sum(dim=1), 0)
        o, cu = zeros(kept, H, D, dtype=_DTYPES[case["out"]]), cu.to(DEV)
        call = binding.prepare_attn_strided(qkv[:, 0], qkv[:, 1], qkv[:, 2], o, cu, N, scale)
        return {"kind": kind, "call": call, "o": o}
    if kind == "padded":
        q, k, v = (_randn(gen, case["dtype"], B, N, H, D) for _ in range(3))
        o = zeros(B, N, H, D, dtype=_DTYPES[case["out"]])
        return {"kind": kind, "call": binding.prepare_attn_padded(q, k, v, o, keep, scale, case["fill"]), "o": o}
    cap = B * N
    q, k, v = (zeros(cap, H, D) for _ in range(3))
    for t in (q, k, v):
        t[:kept] = _randn(gen, case["dtype"], kept, H, D)
    s = {"kind": kind, "x": _randn(gen, case["dtype"], B, N, C), "keep": keep, "q": q, "k": k, "v": v, "N": N, "C": C,
         "packed": zeros(cap, C), "cu": zeros(B + 1, dtype=torch.int32), "gidx": zeros(cap, dtype=torch.int32),
         "o": zeros(cap, H, D), "out": zeros(B, N, C), "scale": scale, "fill": case["fill"], "call": None}
    if kind == "step" and not case["eager"]:
        s["call"] = binding.prepare_pack_attn_unpack(s["x"], keep, q, k, v, s["packed"], s["cu"], s["gidx"], s["o"],
                                                     s["out"], scale, case["fill"])
    elif kind == "stages":
        s["call"] = (binding.prepare_pack(s["x"], keep, s["packed"], s["cu"], s["gidx"]),
                     binding.prepare_attn(q, k, v, s["o"], s["cu"], N, scale),
                     binding.prepare_unpack(s["o"].view(cap, C), keep, s["cu"], s["gidx"], s["out"], case["fill"]))
    return s


def run(s):
    kind = s["kind"]
    if kind == "encoder":
        s["graph"].replay()
        # (a nearly tied score may turn a keep bit, which moves rows and every later mask: the class tokens, which
        # have seen all of them, and the first decision are what two runs can be compared by)
        return {"cls": s["obj"].cls, "scores": s["obj"].scores[0], "keep": s["obj"].keep[0]}
    if kind == "blocks":
        s["graph"].replay()
        return {"cls": s["obj"].cls, "x": s["obj"].x, "cu": s["obj"].cu}
    if kind == "prune":
        binding.ragged_token_scores_l2(s["x"], s["scores"])
        binding.ragged_keep_topk(s["scores"], s["k"], s["keep"])
        binding.ragged_pack(s["x"], s["keep"], s["packed"], s["cu"], s["gidx"])
        binding.ragged_unpack(s["packed"], s["keep"], s["cu"], s["gidx"], s["out"], 1)
        return {n: s[n] for n in ("scores", "keep", "packed", "cu", "gidx", "out")}
    if kind in ("attn", "padded"):
        s["call"]()
        return s["o"]
    if kind == "stages":
        for call in s["call"]:
            call()
    elif s["call"] is not None:
        s["call"]()
    else:
        binding.ragged_pack_attn_unpack(s["x"], s["keep"], s["q"], s["k"], s["v"], s["packed"], s["cu"], s["gidx"],
                                        s["o"], s["out"], s["scale"], s["fill"])
    return {n: s[n] for n in ("packed", "cu", "gidx", "o", "out")}


def work(case):
    kind, B, N, H = case["kind"], case["B"], case["N"], case["H"]
    C = H * D
    row = 2 * C
    n = 1 + (N - 1) * case["keep"]                                    # expected tokens kept per image
    n2 = n * n + (N - 1) * case["keep"] * (1 - case["keep"])          # expected square
    T = B * n
    attn_flops = 4 * C * B * n2
    weights = 12 * C * C * 2 + 13 * C * 2                             # one block (shared by all blocks here)
    if kind == "attn":
        return {"bytes": T * (3 * row + C * _DTYPES[case["out"]].itemsize) + 4 * (B + 1), "flops": attn_flops}
    if kind == "padded":
        out = C * _DTYPES[case["out"]].itemsize
        return {"bytes": B * N + 3 * T * row + (B * N if case["fill"] else T) * out, "flops": attn_flops}
    if kind in ("step", "stages"):
        # x, q, k, v and the mask in; packed, o, out and the indexes out
        return {"bytes": B * N + 4 * T * row + 2 * T * row + (B * N if case["fill"] else T) * row + 4 * T + 4 * (B + 1),
                "flops": attn_flops}
    if kind == "prune":
        T = B * _kept(case)
        return {"bytes": B * N * row + 8 * B * N + B * N + T * row + B * N * row + 4 * T + 4 * (B + 1), "flops": 2 * B * N * C}
    if kind == "blocks":
        return {"bytes": B * N + 2 * T * row + weights + B * row, "flops": case["depth"] * (24 * T * C * C + attn_flops)}
    flops, length = 0, N
    for blk in range(case["depth"]):
        if blk in _prune_at(case):
            length = max(1, int(round(case["keep"] * length)))
        flops += 24 * B * length * C * C + 4 * C * B * length * length
    return {"bytes": B * N * row + weights + B * row, "flops": flops}


def tolerance(case):
    """About four times what the package differs by from the same path with fp32 sums in another order and 16-bit
    roundings at the same places (blocks: 6e-4 in f16, 4e-3 in bf16; encoders 2.6e-3; attention in f16 2.7e-4)."""
    if case["kind"] == "prune":
        return {"rel": 1e-12}                                         # fp64 sums in another order; rows are bit copies
    bf16 = case["dtype"] == "bf16"
    if case["kind"] == "encoder":
        return {"rel": 1e-2, "differ": 0.003}                         # nearly tied scores: 6e-4 of the bits seen to turn
    if case["kind"] == "blocks":
        return {"rel": 1.7e-2 if bf16 else 2.4e-3}
    # bf16: the probabilities carry 16 bits, so results differ by an occasional last place of the output (9e-5)
    return {"rel": 1e-3, "max": 0.04} if bf16 else {"rel": 1.1e-3}
