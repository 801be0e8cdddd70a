"""Launches that start with pairs of whole query tiles (512 rows a workgroup): the rule that counts the pairs against
the same rule written out here, and rows of pairs, of the single tiles behind them and of cut tiles: bit for bit what a
launch of few heads gives (which has no pairs), and against the fp64 oracle."""
import math
import os
import random
import subprocess

import numpy as np
import pytest

from synth import bf16_bits_to_f32, f32_to_bf16_bits, gen_qkv
from tests.util import LSE_REL, REL_L2, assert_close, cut_row_mask, tail_plan, to_dev_bf16

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2511_12056_amd", "csrc")
CLANG = "/opt/rocm/llvm/bin/clang++"
MAIN = r"""
#include "attn_internal.h"
#include <stdio.h>
int main() {
    long long Sq, n_v;
    int BH, n_cu;
    while (scanf("%d %lld %lld %d", &BH, &Sq, &n_v, &n_cu) == 4) {
        const auto w = pda::wide_plan(pda::plan_tail(Sq, BH, n_v, n_cu), n_v, n_cu);
        printf("%d %d\n", w.items, w.odd_heads);
    }
}
"""


def wide_plan(BH, Sq, n_v, n_cu):
    """(pairs, heads whose last of an odd number of tiles is left out): each CU's whole tiles in twos, as far as the
    heads have pairs; none below 224 keys or one round of whole tiles."""
    plan = tail_plan(BH, Sq, n_v, 128, n_cu)
    whole, per_head = plan["n_tiles"] - plan["n_cut"], -(-Sq // 256)
    if n_v < 224 or whole < n_cu or per_head < 2:
        return 0, 0
    wanted = sum((whole // n_cu + (cu < whole % n_cu)) // 2 for cu in range(n_cu))
    have = sum(min(per_head, whole - h * per_head) // 2 for h in range(BH) if whole > h * per_head)
    n = min(wanted, have)
    return n, n // (per_head // 2) if per_head % 2 else 0


def test_rule(tmp_path):
    if not os.path.exists(CLANG):
        pytest.skip("no ROCm clang++ here")
    src, exe = tmp_path / "wide.cpp", tmp_path / "wide"
    src.write_text(MAIN)
    subprocess.run([CLANG, "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I", CSRC, str(src), "-o", str(exe)],
                   check=True, timeout=120)
    rng = random.Random(512)
    cases = [(3, 119056, 119056, 256), (24, 4797, 4701, 256), (24, 9600, 223, 256), (256, 256, 5000, 256), (200, 700, 300, 256)]
    for n_cu in (256, 256, 304, 64, 1):
        for _ in range(800):
            per_head = rng.choice([1, 2, 3, 5, 8, rng.randint(1, 100)])
            BH = max(1, round(n_cu * rng.choice([1, 2, 3, 1.5, rng.uniform(0, 7)]) / per_head))
            cases.append((BH, per_head * 256 - rng.randint(0, 255), rng.choice([rng.randint(200, 3000), rng.randint(1, 120000)]), n_cu))
    out = subprocess.run([str(exe)], input="\n".join(" ".join(map(str, c)) for c in cases), capture_output=True, text=True, check=True, timeout=120)
    got = [tuple(map(int, l.split())) for l in out.stdout.splitlines()]
    assert got == [wide_plan(*c) for c in cases]
    assert got[:5] == [(512, 0), (200, 22), (0, 0), (0, 0), (200, 200)]


def _n_cu():
    import torch
    return torch.cuda.get_device_properties(0).multi_processor_count


def _launch(entry, q, k, v, scale, n_v):
    import torch
    import paper_2511_12056_amd as pda
    B, H, Sq, d = q.shape
    out = torch.full((B, H, Sq, d), float("nan"), device="cuda", dtype=torch.bfloat16 if entry == "bf16" else torch.float32)
    lse = torch.full((B, H, Sq), float("nan"), device="cuda")
    if entry == "base2":
        pda.attn_fwd_base2(q, k, v, out, lse, n_v)
    else:
        (pda.attn_fwd_bf16out if entry == "bf16" else pda.attn_fwd)(q, k, v, out, lse, scale, n_v)
    torch.cuda.synchronize()
    return out, lse


def _scaled(qb, entry, d):
    """Q bits and the scale of the call and of the oracle: for base 2 the scale is folded into Q."""
    if entry != "base2":
        return qb, d ** -0.5
    return f32_to_bf16_bits(bf16_bits_to_f32(qb) * np.float32(d ** -0.5 * math.log2(math.e))), math.log(2.0)


def _repeat(t, H):
    import torch
    return t[:, torch.arange(H, device="cuda") % t.shape[1]].contiguous()


@pytest.mark.gpu
@pytest.mark.parametrize("d", [128, 64])
@pytest.mark.parametrize("H,Sq,n_v", [(135, 1000, 224), (300, 512, 225), (104, 1281, 255), (104, 1281, 256), (180, 700, 257), (180, 700, 287), (180, 700, 288),
                                      (400, 300, 319), (104, 1281, 321), (135, 1000, 353), (135, 1000, 385), (55, 2305, 417), (55, 2305, 449), (30, 4609, 1000)])
def test_every_row_as_in_a_launch_of_few_heads(H, Sq, n_v, d):
    """Even and odd numbers of tiles per head, last tiles of one row to 256, whole and ragged key tiles, every position of
    the last key tile in the ring of buffers; keys beyond n_v are NaN."""
    import torch
    from oracle import attention
    base = 3
    if _n_cu() == 256:
        assert wide_plan(H, Sq, n_v, 256)[0] > 0 and wide_plan(base, Sq, n_v, 256)[0] == 0
        assert tail_plan(base, Sq, n_v, d, 256)["n_cut"] == 0 and tail_plan(H, Sq, n_v, d, 256)["n_cut"] == 0
    qb, kb, vb = gen_qkv(600 + n_v, 1, base, Sq, n_v, d, unit_rms=True)
    pad = torch.full((1, base, 70, d), float("nan"), device="cuda", dtype=torch.bfloat16)
    for entry in ("fp32", "bf16", "base2"):
        eb, scale = _scaled(qb, entry, d)
        q, k, v = to_dev_bf16(eb), torch.cat([to_dev_bf16(kb), pad], 2), torch.cat([to_dev_bf16(vb), pad], 2)
        o, l = _launch(entry, q, k, v, scale, n_v)
        out, lse = _launch(entry, _repeat(q, H), _repeat(k, H), _repeat(v, H), scale, n_v)
        assert torch.equal(out, _repeat(o, H)) and torch.equal(lse, _repeat(l, H)), entry
        if entry != "bf16":
            ro, rl = attention(eb[:, :1], kb[:, :1], vb[:, :1], scale)
            assert_close(out[:, :1].cpu().numpy(), lse[:, :1].cpu().numpy(), ro, rl, f"{(H, Sq, n_v, d)} {entry}")


@pytest.mark.gpu
@pytest.mark.parametrize("entry", ["fp32", "bf16", "base2"])
@pytest.mark.parametrize("B,H,Sq,n_v,d", [(1, 25, 5300, 1700, 128), (1, 25, 5300, 1700, 64), (2, 14, 4900, 2222, 128), (2, 23, 4500, 1601, 64)])
def test_pairs_singles_and_cut_tiles(B, H, Sq, n_v, d, entry):
    """Two and three rounds of whole tiles and some cut ones; two batches.  Sampled rows of every head against the oracle,
    heads of the same content bit for bit where both lie in whole tiles."""
    import torch
    from oracle import attention_head
    base = 5
    if _n_cu() == 256:
        assert wide_plan(B * H, Sq, n_v, 256)[0] > 0 and tail_plan(B * H, Sq, n_v, d, 256)["n_cut"] > 0
    qb, kb, vb = gen_qkv(1400 + n_v, 1, base, Sq, n_v, d, unit_rms=True)
    qb, scale = _scaled(qb, entry, d)
    q, k, v = (_repeat(to_dev_bf16(t), B * H).reshape(B, H, -1, d) for t in (qb, kb, vb))
    out, lse = _launch(entry, q, k, v, scale, n_v)
    out, lse = out.reshape(B * H, Sq, d), lse.reshape(B * H, Sq)
    cut = cut_row_mask(B, H, Sq, n_v, d, _n_cu()).reshape(B * H, Sq)
    rng = np.random.default_rng(n_v)
    rows = np.unique(np.concatenate([[0, 31, 32, 63, 64, 255, 256, 511, 512, Sq - 1], rng.choice(Sq, size=50, replace=False)]))
    dr = torch.from_numpy(rows).cuda()
    want = [attention_head(qb[0, i], kb[0, i], vb[0, i], scale, n_v, rows=rows) for i in range(base)]
    first = {}
    for h in range(B * H):
        o, l = out[h][dr].float().cpu().numpy(), lse[h][dr].cpu().numpy()
        ro, rl = want[h % base]
        tol = REL_L2 + (2.0 ** -9 / np.sqrt(3.0) if entry == "bf16" else 0.0)
        assert np.isfinite(o).all() and np.sqrt(((o - ro) ** 2).sum() / (ro ** 2).sum()) <= tol, h
        assert (np.abs(l - rl) / np.maximum(np.abs(rl), 1.0)).max() <= LSE_REL, h
        whole = torch.from_numpy(~cut[h]).cuda()
        fo, fl, fw = first.setdefault(h % base, (out[h], lse[h], whole))
        both = whole & fw
        assert torch.equal(out[h][both], fo[both]) and torch.equal(lse[h][both], fl[both]), h


@pytest.mark.gpu
@pytest.mark.parametrize("entry", ["fp32", "bf16", "base2"])
@pytest.mark.parametrize("d,H,every", [(128, 140, 3), (64, 140, 1), (64, 1300, 1), (128, 1300, 2)])
def test_tiles_given_back(d, H, every, entry):
    """Rows that need the second sweep in pairs: one row of either tile, or all rows; in so many pairs that a workgroup's
    list of sixteen tiles is full (1 300 heads x 1 000 rows: ten pairs for every workgroup).  Rows beside them keep their bits."""
    import torch
    from oracle import attention
    base, Sq, n_v = 6, 1000, 300
    if _n_cu() == 256:
        assert wide_plan(H, Sq, n_v, 256)[0] > 0
    rng = np.random.default_rng(d + H)
    q = rng.standard_normal((1, base, Sq, d)).astype(np.float32)
    k = (rng.standard_normal((1, base, n_v, d)) * 0.05).astype(np.float32)
    v = rng.standard_normal((1, base, n_v, d)).astype(np.float32)
    row = {0: 250, 1: 290, 2: 999, 3: 5, 4: 767, 5: 512}
    for h in range(0, base, every):
        k[0, h, 200 + h] = q[0, h, row[h]] * np.float32(1.5 * 128 / d)          # > 64 log2 units above the first tile
    if every == 1:
        k[0, 3 if H < 1000 else slice(None), 150:] *= np.float32(600.0)         # every row, of every head: two tiles of each pair
    qb, kb, vb = (f32_to_bf16_bits(x) for x in (q, k, v))
    scale, oracle_scale = 1.0, 1.0
    if entry == "base2":
        qb, oracle_scale = f32_to_bf16_bits(q * np.float32(math.log2(math.e))), math.log(2.0)
    dq, dk, dv = to_dev_bf16(qb), to_dev_bf16(kb), to_dev_bf16(vb)
    o, l = _launch(entry, dq, dk, dv, scale, n_v)
    out, lse = _launch(entry, _repeat(dq, H), _repeat(dk, H), _repeat(dv, H), scale, n_v)
    for h in range(H):
        assert torch.equal(out[0, h], o[0, h % base]) and torch.equal(lse[0, h], l[0, h % base]), h
    ro, rl = attention(qb, kb, vb, oracle_scale)
    o, l = o.float().cpu().numpy().astype(np.float64), l.cpu().numpy()
    tol = REL_L2 + (2.0 ** -9 / np.sqrt(3.0) if entry == "bf16" else 0.0)
    assert np.isfinite(o).all() and np.sqrt(((o - ro) ** 2).sum() / (ro ** 2).sum()) <= tol
    assert (np.abs(l - rl) / np.maximum(np.abs(rl), 1.0)).max() <= LSE_REL


@pytest.mark.gpu
def test_views_and_replays_of_a_captured_launch():
    import torch
    import paper_2511_12056_amd as pda
    B, H, S, d, a, b = 2, 70, 1500, 128, 130, 1203
    if _n_cu() == 256:
        assert wide_plan(B * (H - 2), b - a, 301, 256)[0] > 0
    gen = torch.Generator(device="cuda").manual_seed(8)
    q, k, v = (torch.randn(B, H, S, d, generator=gen, device="cuda").to(torch.bfloat16) for _ in range(3))
    qs, ks, vs = q[:, 1:-1, a:b], k[:, 1:-1, 64:365], v[:, 1:-1, 64:365]
    want, wl = _launch("fp32", qs.contiguous(), ks.contiguous(), vs.contiguous(), 0.1, 301)
    out, lse = torch.zeros(B, H, S, d, device="cuda"), torch.zeros(B, H, S, device="cuda")
    st = torch.cuda.Stream()
    st.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(st):
        pda.attn_fwd_strided(qs, ks, vs, out[:, 1:-1, a:b], lse[:, 1:-1, a:b], 0.1)
        st.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=st):
            pda.attn_fwd_strided(qs, ks, vs, out[:, 1:-1, a:b], lse[:, 1:-1, a:b], 0.1)
        for _ in range(3):
            out.zero_()
            lse.zero_()
            graph.replay()
            st.synchronize()
            assert torch.equal(out[:, 1:-1, a:b], want) and torch.equal(lse[:, 1:-1, a:b], wl)
            out[:, 1:-1, a:b] = 0
            lse[:, 1:-1, a:b] = 0
            assert not out.any() and not lse.any()             # nothing beside the view was written
