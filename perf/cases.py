"""The workloads the attention library is measured on: calls of its public entry points as a video
diffusion transformer's inference loop makes them, from one tiny launch to the 720p x 129-frame
head-chunk pipeline.

A case is a dict with a "kind" (which entry points a pass goes through) and the sizes of that kind:

    attn       pda_attn_fwd             B, H, Sq, Skv, valid (keys not masked), d
    bf16out    pda_attn_fwd_bf16out     the same, result in bf16 for the next projection
    pipeline   pda_headchunk_run_ex     H heads over S tokens in groups of `group` heads, hand-off into
                                        the head-major or the final token-major layout
    split      pda_attn_fwd_strided     H heads, keys in `chunks` views of one tensor, and the exact merge
               + pda_attn_merge         of the partial results (co-processing shares)
    packed     pda_pack_heads (x3)      fp32 projections to bf16 heads with the softmax scale folded into
               + pda_attn_fwd_base2     Q, then attention on exponents of 2
    post       pda_pipesp_postprocess   head order of the exchanges -> head order of the model, fp32

Inputs are unit-RMS Gaussian vectors (what a normalised Q and K are), made on the GPU from the seed.
"""
from __future__ import annotations

import math

import torch

import paper_2511_12056_amd as pda

LOG2E = math.log2(math.e)
LARGEST_FLOPS = 4.0 * 119056 * 119056 * 128 * 24     # the 720p pipeline

_streams = {}


def _pipeline_streams():
    """The compute and the drain stream of a program: made once, as such a program keeps them."""
    dev = torch.cuda.current_device()
    if dev not in _streams:
        _streams[dev] = (torch.cuda.Stream(), torch.cuda.Stream())
    return _streams[dev]


def listed():
    return [
        # the smallest call: 2 heads of a 4 x 16 x 16 latent grid; latency and launches
        {"name": "tiny_d64", "kind": "attn", "B": 1, "H": 2, "Sq": 1024, "Skv": 1024, "valid": 1024, "d": 64},
        # one head of a short clip (8 x 30 x 40 latent grid): the unit of a head-by-head pipeline
        {"name": "one_head_clip", "kind": "attn", "B": 1, "H": 1, "Sq": 9600, "Skv": 9600, "valid": 9600, "d": 128},
        # all 24 heads of that clip in one launch
        {"name": "lowres_clip", "kind": "attn", "B": 1, "H": 24, "Sq": 9600, "Skv": 9600, "valid": 9600, "d": 128},
        # three heads at 544 x 960 x 129 frames with 256 text tokens, 100 of them padding
        {"name": "group_544x960", "kind": "attn", "B": 1, "H": 3, "Sq": 67576, "Skv": 67576, "valid": 67476, "d": 128},
        # many queries on few keys, a masked tail: attention to a short conditioning sequence
        {"name": "few_keys", "kind": "attn", "B": 1, "H": 24, "Sq": 16384, "Skv": 600, "valid": 570, "d": 128},
        # head dimension 64 on a long sequence
        {"name": "long_d64", "kind": "attn", "B": 1, "H": 6, "Sq": 67576, "Skv": 67576, "valid": 67576, "d": 64},
        # a batch of two (guidance), ragged length, the result in bf16
        {"name": "batch_bf16out", "kind": "bf16out", "B": 2, "H": 12, "Sq": 4797, "Skv": 4797, "valid": 4701, "d": 128},
        # a short sequence head by head: 24 launches with their hand-offs, bound by their number
        {"name": "pipeline_short", "kind": "pipeline", "H": 24, "S": 2048, "d": 128, "group": 1, "token_major": True},
        # the flagship: 24 heads at 720p x 129 frames in groups of three, head-major hand-off
        {"name": "pipeline_720p", "kind": "pipeline", "H": 24, "S": 119056, "d": 128, "group": 3, "token_major": False},
        # six heads at 720p as four key chunks with their merge
        {"name": "split_merge_720p", "kind": "split", "H": 6, "S": 119056, "d": 128, "chunks": 4},
        # from the fp32 projections of the short clip to its attention
        {"name": "packed_clip", "kind": "packed", "H": 24, "S": 9600, "d": 128},
        # the reordering after the exchanges of eight ranks with three heads each, at 720p
        {"name": "post_720p", "kind": "post", "rows": 119056, "h": 3, "n": 8, "d": 128},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["attn", "attn", "attn", "bf16out", "pipeline", "split", "packed", "post"])
    d = rng.choice([128, 128, 64])
    while True:
        if kind in ("attn", "bf16out"):
            s = _log_int(rng, 300, 119056)
            skv = rng.choice([s, s, s, _log_int(rng, 100, 119056)])
            case = {"kind": kind, "B": rng.choice([1, 1, 2]), "H": rng.randint(1, 24), "Sq": s, "Skv": skv,
                    "valid": skv - rng.choice([0, rng.randint(0, 99)]), "d": d}
        elif kind == "pipeline":
            H = rng.choice([6, 12, 24])
            case = {"kind": kind, "H": H, "S": _log_int(rng, 1000, 67576), "d": d, "group": rng.choice([1, 2, 3]),
                    "token_major": rng.random() < 0.5}
        elif kind == "split":
            case = {"kind": kind, "H": rng.randint(1, 12), "S": _log_int(rng, 2000, 119056), "d": d, "chunks": rng.randint(2, 8)}
        elif kind == "packed":
            case = {"kind": kind, "H": rng.randint(1, 24), "S": _log_int(rng, 1000, 67576), "d": d}
        else:
            case = {"kind": kind, "rows": _log_int(rng, 1000, 119056), "h": rng.randint(1, 8), "n": rng.randint(2, 8), "d": d}
        if work(case)["flops"] <= LARGEST_FLOPS / 4:
            return case


def _unit_rms(gen, *shape):
    """bf16 Gaussian tensor whose last-axis vectors have RMS one."""
    x = torch.randn(*shape, generator=gen, device="cuda")
    x *= x.square().mean(dim=-1, keepdim=True).rsqrt_()
    return x.to(torch.bfloat16)


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    kind, d = case["kind"], case["d"]
    f32 = dict(device="cuda", dtype=torch.float32)
    st = {"case": case, "scale": d ** -0.5}
    if kind in ("attn", "bf16out"):
        B, H, Sq, Skv = case["B"], case["H"], case["Sq"], case["Skv"]
        st["q"], st["k"], st["v"] = _unit_rms(gen, B, H, Sq, d), _unit_rms(gen, B, H, Skv, d), _unit_rms(gen, B, H, Skv, d)
        st["out"] = torch.empty(B, H, Sq, d, device="cuda", dtype=torch.float32 if kind == "attn" else torch.bfloat16)
        st["lse"] = torch.empty(B, H, Sq, **f32)
    elif kind == "pipeline":
        H, S = case["H"], case["S"]
        st["q"], st["k"], st["v"] = (_unit_rms(gen, 1, H, S, d) for _ in range(3))
        st["out"], st["lse"] = torch.empty(1, H, S, d, **f32), torch.empty(1, H, S, **f32)
        st["sink"] = torch.empty((1, S, H, d) if case["token_major"] else (1, H, S, d), **f32)
        st["groups"] = [case["group"]] * (H // case["group"])
        st["streams"] = _pipeline_streams()
    elif kind == "split":
        H, S, n = case["H"], case["S"], case["chunks"]
        st["q"], st["k"], st["v"] = (_unit_rms(gen, 1, H, S, d) for _ in range(3))
        cuts = [S * i // n for i in range(n + 1)]
        st["chunks"] = [(st["k"][:, :, a:b], st["v"][:, :, a:b]) for a, b in zip(cuts, cuts[1:])]
        st["parts"] = [(torch.empty(1, H, S, d, **f32), torch.empty(1, H, S, **f32)) for _ in range(n)]
        st["out"], st["lse"] = torch.empty(1, H, S, d, **f32), torch.empty(1, H, S, **f32)
    elif kind == "packed":
        H, S = case["H"], case["S"]
        st["x"] = [torch.randn(1, S, H, d, generator=gen, device="cuda") for _ in range(3)]
        st["qkv"] = [torch.empty(1, H, S, d, device="cuda", dtype=torch.bfloat16) for _ in range(3)]
        st["out"], st["lse"] = torch.empty(1, H, S, d, **f32), torch.empty(1, H, S, **f32)
    else:
        rows, h, n = case["rows"], case["h"], case["n"]
        st["arrived"] = torch.randn(rows, h * n, d, generator=gen, device="cuda")
        st["hidden"] = torch.empty(rows, n * h, d, **f32)
    return st


def run(st):
    case = st["case"]
    kind = case["kind"]
    if kind == "attn":
        return pda.attn_fwd(st["q"], st["k"], st["v"], st["out"], st["lse"], st["scale"], case["valid"])
    if kind == "bf16out":
        return pda.attn_fwd_bf16out(st["q"], st["k"], st["v"], st["out"], st["lse"], st["scale"], case["valid"])
    if kind == "pipeline":
        cs, ds = st["streams"]
        here = torch.cuda.current_stream()
        cs.wait_stream(here)                  # the projections that made q, k and v
        ds.wait_stream(here)                  # whoever still reads the last hand-off
        pda.headchunk_run_ex(st["q"], st["k"], st["v"], st["out"], st["lse"], st["scale"], st["groups"], cs, ds,
                             sink=st["sink"],
                             sink_layout=pda.PDA_SINK_TOKEN_FINAL if case["token_major"] else pda.PDA_SINK_HEAD_MAJOR)
        here.wait_stream(cs)
        here.wait_stream(ds)
        return st["out"], st["lse"], st["sink"]
    if kind == "split":
        for (k, v), (o, l) in zip(st["chunks"], st["parts"]):
            pda.attn_fwd_strided(st["q"], k, v, o, l, st["scale"])
        pda.attn_merge([o for o, _ in st["parts"]], [l for _, l in st["parts"]], st["out"], st["lse"])
        return st["out"], st["lse"], st["parts"]
    if kind == "packed":
        q, k, v = st["qkv"]
        pda.pack_heads(st["x"][0], q, True, premul=st["scale"] * LOG2E)
        pda.pack_heads(st["x"][1], k, True)
        pda.pack_heads(st["x"][2], v, False)
        pda.attn_fwd_base2(q, k, v, st["out"], st["lse"])
        return q, k, v, st["out"], st["lse"]
    return pda.pipesp_postprocess(st["arrived"], case["h"], case["n"], st["hidden"])


def _exact_attn(q, k, v, scale, valid):
    """softmax(scale q k^T) v and its log-sum-exp in 64 bits, [B,H,Sq,d] and [B,H,Sq], by blocks of queries."""
    B, H, Sq, d = q.shape
    out = torch.empty(B, H, Sq, v.shape[-1], device=q.device, dtype=torch.float64)
    lse = torch.empty(B, H, Sq, device=q.device, dtype=torch.float64)
    step = max(1, min(Sq, (1 << 27) // max(1, valid)))
    for b in range(B):
        for h in range(H):
            kt = k[b, h, :valid].double().t().contiguous()
            vv = v[b, h, :valid].double()
            for r in range(0, Sq, step):
                s = torch.mm(q[b, h, r:r + step].double() * scale, kt)
                l = torch.logsumexp(s, dim=-1)
                out[b, h, r:r + step] = torch.mm(s.sub_(l[:, None]).exp_(), vv)
                lse[b, h, r:r + step] = l
    return out, lse


EXACT_FLOPS = 6e13     # what the 64-bit calculation does in well under 20 seconds


def exact(case, seed):
    """What `run` returns, in 64 bits; bf16 tensors that a later call of the pass reads are taken as that
    call gets them, so each output stands for its own entry point."""
    if work(case)["flops"] > EXACT_FLOPS:
        return None
    st = prepare(case, seed)
    kind, scale = case["kind"], st["scale"]
    if kind in ("attn", "bf16out"):
        return _exact_attn(st["q"], st["k"], st["v"], scale, case["valid"])
    if kind == "pipeline":
        out, lse = _exact_attn(st["q"], st["k"], st["v"], scale, case["S"])
        return out, lse, out.transpose(1, 2).contiguous() if case["token_major"] else out
    if kind == "split":
        parts = [_exact_attn(st["q"], k, v, scale, k.shape[2]) for k, v in st["chunks"]]
        lses = torch.stack([l for _, l in parts])
        lse = torch.logsumexp(lses, dim=0)
        out = torch.zeros_like(parts[0][0])
        for (o, l) in parts:
            out += o * (l - lse).exp()[..., None]
        return out, lse, parts
    if kind == "packed":
        rms = [x.double().square().mean(dim=-1, keepdim=True).rsqrt() for x in st["x"][:2]]
        q = (st["x"][0].double() * rms[0] * (scale * LOG2E)).transpose(1, 2)
        k = (st["x"][1].double() * rms[1]).transpose(1, 2)
        v = st["x"][2].double().transpose(1, 2)
        qr, kr, vr = (t.float().to(torch.bfloat16) for t in (q, k, v))
        return (q.contiguous(), k.contiguous(), v.contiguous(), *_exact_attn(qr, kr, vr, math.log(2.0), case["S"]))
    rows, h, n, d = case["rows"], case["h"], case["n"], case["d"]
    return st["arrived"].double().view(rows, h, n, d).transpose(1, 2).reshape(rows, n * h, d)


def work(case):
    """Each input read once, each result written once; 4 Sq Skv d operations per head."""
    kind, d = case["kind"], case["d"]
    if kind in ("attn", "bf16out"):
        bh, Sq, n = case["B"] * case["H"], case["Sq"], case["valid"]
        out = 4 if kind == "attn" else 2
        return {"bytes": bh * (Sq * d * (2 + out) + 2 * n * d * 2 + Sq * 4), "flops": 4.0 * bh * Sq * n * d}
    if kind == "post":
        return {"bytes": 2.0 * case["rows"] * case["h"] * case["n"] * d * 4, "flops": 0}
    H, S = case["H"], case["S"]
    flops = 4.0 * H * S * S * d
    attn = H * S * (3 * d * 2 + d * 4 + 4)
    if kind == "pipeline":
        return {"bytes": attn + H * S * d * 4, "flops": flops}
    if kind == "split":
        return {"bytes": attn + case["chunks"] * H * S * (d + 1) * 4, "flops": flops}
    return {"bytes": attn + H * S * 3 * d * 6, "flops": flops}


def tolerance(case):
    """Four times what the path differs from the same attention in 64 bits (1.7e-3 in the 2-norm at every
    size: the rounding of the probabilities to bf16); a result in bf16 adds its own rounding.  The
    reordering moves values."""
    if case["kind"] == "post":
        return "exact"
    return {"rel": 8e-3 if case["kind"] == "bf16out" else 7e-3}
