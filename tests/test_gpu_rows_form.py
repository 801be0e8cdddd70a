"""Launches of few query rows, whose workgroups finish 32 or 64 rows each and share the keys among eight wavefronts: the
rule that picks them against the same rule written out here, and their results at the edges of row blocks, key tiles
and key shares against the fp64 oracle."""
import math
import os
import random
import subprocess

import numpy as np
import pytest

from synth import bf16_bits_to_f32, f32_to_bf16_bits, gen_qkv
from tests.util import assert_close, tail_plan, to_dev_bf16

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2511_12056_amd", "csrc")
CLANG = "/opt/rocm/llvm/bin/clang++"
MAIN = r"""
#include "attn_internal.h"
#include <stdio.h>
int main() {
    long long Sq, n_v;
    int BH, d, n_cu;
    while (scanf("%d %lld %lld %d %d", &BH, &Sq, &n_v, &d, &n_cu) == 5)
        printf("%d\n", pda::rows_form(pda::plan_tail(Sq, BH, n_v, n_cu), Sq, BH, n_v, d, n_cu));
}
"""


def rows_form(BH, Sq, n_v, d, n_cu):
    """Every tile of the plan is cut, and the keys do not exceed what blocks of 32 rows (in rounds of n_cu) allow."""
    plan = tail_plan(BH, Sq, n_v, d, n_cu)
    if plan["split"] < 2 or plan["n_cut"] != plan["n_tiles"]:
        return False
    rounds = -(-Sq // 32) * BH / n_cu
    if d == 64:
        if rounds <= 2:
            return n_v <= (3072 if rounds < 1 / 4 else 6144 if 3 / 8 <= rounds <= 1 else 4096)
        return n_v <= (2048 if rounds <= 3 else 1536 if rounds <= 4 else 0)
    if rounds <= 1:
        return n_v <= (2048 if rounds < 1 / 4 else 3072 if rounds < 1 / 2 else 5120)
    return n_v <= (4096 if rounds <= 2 else 1152 if rounds < 3.5 else 1536 if rounds <= 4 else 0)


def test_rule(tmp_path):
    if not os.path.exists(CLANG):
        pytest.skip("no ROCm clang++ here")
    src, exe = tmp_path / "rows.cpp", tmp_path / "rows"
    src.write_text(MAIN)
    subprocess.run([CLANG, "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I", CSRC, str(src), "-o", str(exe)],
                   check=True, timeout=120)
    rng = random.Random(32)
    cases = [(2, 1024, 1024, 64, 256), (2, 1024, 1023, 64, 256), (1, 2048, 2048, 128, 256), (1, 2047, 3072, 128, 256), (1, 2016, 3072, 128, 256)]
    for n_cu in (256, 256, 256, 304, 64, 1):
        for _ in range(1500):
            Sq = rng.randint(1, 3000)
            BH = max(1, round(n_cu * rng.choice([0.1, 0.25, 0.375, 0.5, 1, 2, 3, 3.5, 4, rng.uniform(0, 5)]) / -(-Sq // 32)))
            cases.append((BH, Sq, rng.choice([rng.randint(900, 7000), rng.choice([1024, 1152, 1536, 2048, 3072, 4096, 5120, 6144]) + rng.randint(0, 1)]),
                          rng.choice([64, 128]), n_cu))
    out = subprocess.run([str(exe)], input="\n".join(" ".join(map(str, c)) for c in cases), capture_output=True, text=True, check=True, timeout=120)
    got = [bool(int(x)) for x in out.stdout.split()]
    assert got == [rows_form(*c) for c in cases]
    assert got[:5] == [True, False, True, True, False] and 0.1 < got.count(True) / len(got) < 0.9


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


@pytest.mark.gpu
@pytest.mark.parametrize("d", [128, 64])
@pytest.mark.parametrize("B,H,Sq,n_v", [(1, 1, 1, 1024), (1, 2, 31, 1025), (2, 1, 32, 1055), (1, 3, 33, 1056), (1, 1, 63, 1087), (2, 2, 65, 1281),
                                        (1, 3, 97, 1500), (1, 5, 301, 2017), (3, 3, 800, 2048),
                                        (3, 5, 799, 1100), (1, 9, 1025, 1311), (2, 12, 1000, 1024)])
def test_edges_against_the_oracle(B, H, Sq, n_v, d):
    """Rows and keys at the edges of blocks, shares of unequal length, keys beyond kv_valid_len that must not be read."""
    import torch
    from oracle import attention
    if _n_cu() == 256:
        assert rows_form(B * H, Sq, n_v, d, 256)
    qb, kb, vb = gen_qkv(9000 + Sq + n_v, B, H, Sq, n_v, d, unit_rms=True)
    q, k, v = to_dev_bf16(qb), to_dev_bf16(kb), to_dev_bf16(vb)
    pad = torch.full((B, H, 77, d), float("nan"), device="cuda", dtype=torch.bfloat16)
    k, v = torch.cat([k, pad], 2).contiguous(), torch.cat([v, pad], 2).contiguous()
    ro, rl = attention(qb, kb, vb, d ** -0.5)
    out, lse = _launch("fp32", q, k, v, d ** -0.5, n_v)
    assert_close(out.cpu().numpy(), lse.cpu().numpy(), ro, rl, f"{(B, H, Sq, n_v, d)}")
    out16, lse16 = _launch("bf16", q, k, v, d ** -0.5, n_v)
    assert torch.equal(out16, out.to(torch.bfloat16)) and torch.equal(lse16, lse)
    q2b = f32_to_bf16_bits(bf16_bits_to_f32(qb) * np.float32(d ** -0.5 * math.log2(math.e)))
    r2, l2 = attention(q2b, kb, vb, math.log(2.0))
    o, l = _launch("base2", to_dev_bf16(q2b), k, v, None, n_v)
    assert_close(o.cpu().numpy(), l.cpu().numpy(), r2, l2, f"base 2 {(B, H, Sq, n_v, d)}")


@pytest.mark.gpu
@pytest.mark.parametrize("d", [128, 64])
def test_far_apart_scores_and_large_values(d):
    """The reference moves late in a share, a share whose weights vanish against another's, values of 2^100, one row
    whose scores all lie far below the others'; and rows beside such rows."""
    from oracle import attention
    H, Sq, n_v = 4, 70, 1100
    rng = np.random.default_rng(77 + d)
    q = rng.standard_normal((1, H, Sq, d)).astype(np.float32)
    k = (rng.standard_normal((1, H, n_v, d)) * 0.3).astype(np.float32)
    v = rng.standard_normal((1, H, n_v, d)).astype(np.float32)
    k[0, 0, 1090] = q[0, 0, 33] * np.float32(1.5 * 128 / d)       # the last keys of the last share
    k[0, 1, 5] = q[0, 1, 0] * np.float32(3.0 * 128 / d)           # the first share, all others vanish for row 0
    k[0, 2, 600:] *= np.float32(200.0)
    v[0, 2] *= np.float32(2.0 ** 100)
    q[0, 3, 69] *= np.float32(1e-3)
    qb, kb, vb = (f32_to_bf16_bits(x) for x in (q, k, v))
    if _n_cu() == 256:
        assert rows_form(H, Sq, n_v, d, 256)
    out, lse = _launch("fp32", to_dev_bf16(qb), to_dev_bf16(kb), to_dev_bf16(vb), 1.0, n_v)
    ro, rl = attention(qb, kb, vb, 1.0)
    o, l = out.cpu().numpy().astype(np.float64), lse.cpu().numpy()
    assert np.isfinite(o).all() and np.isfinite(l).all()
    for h in range(H):                                            # head by head: head 2 spans 2^100
        assert np.sqrt(((o[0, h] - ro[0, h]) ** 2).sum() / (ro[0, h] ** 2).sum()) <= 1e-2, h
    assert (np.abs(l - rl) / np.maximum(np.abs(rl), 1.0)).max() <= 1e-3


@pytest.mark.gpu
def test_strided_views_and_a_captured_graph():
    """Head and batch strides other than compact ones, and replays of a captured launch."""
    import torch
    import paper_2511_12056_amd as pda
    B, H, S, d, a, b = 2, 5, 1400, 64, 100, 290
    if _n_cu() == 256:
        assert rows_form(B * 2, b - a, 1201, d, 256)
    gen = torch.Generator(device="cuda").manual_seed(3)
    q, k, v = (torch.randn(B, H, S, d, generator=gen, device="cuda").to(torch.bfloat16) for _ in range(3))
    want, wl = _launch("fp32", q[:, 1:3, a:b].contiguous(), k[:, 1:3, 64:1265].contiguous(), v[:, 1:3, 64:1265].contiguous(), 0.1, 1201)
    out, lse = torch.zeros(B, H, S, d, device="cuda"), torch.zeros(B, H, S, device="cuda")

    def call():
        pda.attn_fwd_strided(q[:, 1:3, a:b], k[:, 1:3, 64:1265], v[:, 1:3, 64:1265], out[:, 1:3, a:b], lse[:, 1:3, a:b], 0.1)

    st = torch.cuda.Stream()
    st.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(st):
        call()
        st.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=st):
            call()
        for _ in range(3):
            out.zero_()
            lse.zero_()
            graph.replay()
            st.synchronize()
            assert torch.equal(out[:, 1:3, a:b], want) and torch.equal(lse[:, 1:3, a:b], wl)
            out[:, 1:3, a:b] = 0
            lse[:, 1:3, a:b] = 0
            assert not out.any() and not lse.any()             # nothing beside the view was written


@pytest.mark.gpu
@pytest.mark.parametrize("d", [128, 64])
@pytest.mark.parametrize("ranges", [2, 3, 4, 5])
def test_cut_form_of_few_ranges(ranges, d):
    """The merge of so few key ranges, which the rule leaves to larger launches (variant 3 always takes the cut form)."""
    import torch
    import paper_2511_12056_amd as pda
    from oracle import attention
    Sq, n_v = 201, 512 * ranges + 511
    if _n_cu() == 256:
        assert tail_plan(1, Sq, n_v, d, 256)["split"] == ranges
    qb, kb, vb = gen_qkv(700 + ranges, 1, 1, Sq, n_v, d, unit_rms=True)
    out, lse = torch.full((1, 1, Sq, d), float("nan"), device="cuda"), torch.full((1, 1, Sq), float("nan"), device="cuda")
    pda.attn_fwd_variant(to_dev_bf16(qb), to_dev_bf16(kb), to_dev_bf16(vb), out, lse, d ** -0.5, variant=3)
    assert_close(out.cpu().numpy(), lse.cpu().numpy(), *attention(qb, kb, vb, d ** -0.5), f"{ranges} ranges, d={d}")


@pytest.mark.gpu
@pytest.mark.parametrize("d,n_v", [(128, 1024), (128, 1499), (128, 2047), (64, 1025), (64, 1499)])
@pytest.mark.parametrize("Sq", [993, 1024, 1025])
def test_two_blocks_of_rows_give_the_bits_of_one(Sq, d, n_v):
    """13 heads (more than a round of 32-row blocks: 64 rows a workgroup) against one of them alone."""
    import torch
    if _n_cu() == 256:
        assert rows_form(13, Sq, n_v, d, 256) and rows_form(1, Sq, n_v, d, 256)
    qb, kb, vb = gen_qkv(80 + Sq, 1, 13, Sq, n_v, d, unit_rms=True)
    q, k, v = to_dev_bf16(qb), to_dev_bf16(kb), to_dev_bf16(vb)
    for entry in ("fp32", "bf16"):
        out, lse = _launch(entry, q, k, v, d ** -0.5, n_v)
        for h in (0, 7, 12):
            o, l = _launch(entry, *(t[:, h:h + 1].contiguous() for t in (q, k, v)), d ** -0.5, n_v)
            assert torch.equal(out[:, h], o[:, 0]) and torch.equal(lse[:, h], l[:, 0]), (entry, h)


JOIN = r"""
#include "attn_internal.h"
#include <stdio.h>
int main() {
    long long Sq, n_v;
    int B, d, n_cu, alone, hg, n;
    while (scanf("%d %lld %lld %d %d %d %d %d", &B, &Sq, &n_v, &d, &n_cu, &alone, &hg, &n) == 8) {
        const std::vector<int> sizes(n, hg);
        const auto steps = pda::pipeline_steps(sizes, B, Sq, n_v, n_cu, alone != 0);
        for (const auto& s : pda::join_steps(steps, B, Sq, n_v, d, n_cu, alone != 0)) printf("%d:%d:%d ", s.h0, s.hg, s.groups);
        printf("\n");
    }
}
"""


def test_joined_steps(tmp_path):
    """Steps of a pipeline in one launch: every head once and in order, none beyond six blocks of 32 rows per compute unit
    unless one step is, none joined outside the rule."""
    if not os.path.exists(CLANG):
        pytest.skip("no ROCm clang++ here")
    src, exe = tmp_path / "join.cpp", tmp_path / "join"
    src.write_text(JOIN)
    subprocess.run([CLANG, "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I", CSRC, str(src), "-o", str(exe)],
                   check=True, timeout=120)
    rng = random.Random(24)
    cases = [(1, 2048, 2048, 128, 256, 0, 1, 24), (1, 2048, 2048, 128, 256, 1, 1, 24), (1, 2048, 2049, 128, 256, 0, 1, 24), (1, 2048, 2049, 64, 256, 0, 1, 49),
             (1, 2048, 1000, 64, 256, 0, 1, 24)]
    for _ in range(1500):
        cases.append((rng.randint(1, 2), rng.randint(1, 5000), rng.randint(900, 5000), rng.choice([64, 128]), rng.choice([256, 256, 304, 64]),
                      rng.randint(0, 4) // 4, rng.randint(1, 3), rng.randint(0, 60)))
    out = subprocess.run([str(exe)], input="\n".join(" ".join(map(str, c)) for c in cases), capture_output=True, text=True, check=True, timeout=120)
    rows = [[tuple(map(int, x.split(":"))) for x in l.split()] for l in out.stdout.split("\n")][:len(cases)]
    assert [len(r) for r in rows[:5]] == [1, 24, 3, 3, 1]
    for (B, Sq, n_v, d, n_cu, alone, hg, n), steps in zip(cases, rows):
        assert sum(g for _, _, g in steps) == n and all(h == hg for _, h, _ in steps)
        assert [h0 for h0, _, _ in steps] == [sum(g * hg for _, _, g in steps[:i]) for i in range(len(steps))]
        plan = tail_plan(B * hg, Sq, n_v, d, n_cu)
        items = plan["n_tiles"] + plan["n_cut"] * (plan["split"] - 1)
        alone_fit = n_cu // items if 2 * items <= n_cu else 1               # groups of a launch without joining
        for _, _, g in steps:
            if alone:
                assert g == 1
            elif g > alone_fit:
                assert rows_form(B * hg, Sq, n_v, d, n_cu) and n_v * d <= 2048 * 128 and g * B * hg * -(-Sq // 32) <= 6 * n_cu


@pytest.mark.gpu
@pytest.mark.parametrize("S,n_v,d,groups", [(1100, 1100, 128, [1] * 50), (2000, 2000, 64, [1] * 20 + [2] * 9), (1030, 1025, 128, [3] * 8 + [1])])
def test_joined_launches_of_a_pipeline(S, n_v, d, groups):
    """Each group the bits of its own launch, the hand-off complete; more groups than one launch takes."""
    import torch
    import paper_2511_12056_amd as pda
    H = sum(groups)
    gen = torch.Generator(device="cuda").manual_seed(S)
    q, k, v = (torch.randn(1, H, S, d, generator=gen, device="cuda").to(torch.bfloat16) for _ in range(3))
    ref, rlse = torch.empty(1, H, S, d, device="cuda"), torch.empty(1, H, S, device="cuda")
    h0 = 0
    for g in groups:
        if _n_cu() == 256:
            assert rows_form(g, S, n_v, d, 256)
        sl = slice(h0, h0 + g)
        pda.attn_fwd_strided(q[:, sl], k[:, sl], v[:, sl], ref[:, sl], rlse[:, sl], 0.1, n_v)
        h0 += g
    cs, ds = torch.cuda.Stream(), torch.cuda.Stream()
    for layout in (pda.PDA_SINK_HEAD_MAJOR, pda.PDA_SINK_TOKEN_FINAL):
        out, lse = torch.full_like(ref, float("nan")), torch.full_like(rlse, float("nan"))
        sink = torch.full((1, H, S, d) if layout == pda.PDA_SINK_HEAD_MAJOR else (1, S, H, d), float("nan"), device="cuda")
        torch.cuda.synchronize()
        pda.headchunk_run_ex(q, k, v, out, lse, 0.1, groups, cs, ds, sink_layout=layout, kv_valid_len=n_v, sink=sink)
        cs.synchronize(); ds.synchronize()
        assert torch.equal(out, ref) and torch.equal(lse, rlse)
        assert torch.equal(sink, ref if layout == pda.PDA_SINK_HEAD_MAJOR else ref.transpose(1, 2))
