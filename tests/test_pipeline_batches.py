"""Pipelines of small head groups: several groups share a launch, and each gets the bits it has in a launch
of its own."""
import os
import random
import subprocess

import pytest

from tests.util import tail_plan

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2511_12056_amd", "csrc")
CLANG = "/opt/rocm/llvm/bin/clang++"
MAIN = r"""
#include "attn_internal.h"
#include <stdio.h>
int main() {
    long long Sq, n_v;
    int BH, n_cu, left;
    while (scanf("%d %lld %lld %d %d", &BH, &Sq, &n_v, &n_cu, &left) == 5)
        printf("%d %lld\n", pda::batch_of_groups(Sq, BH, n_v, n_cu, left), (long long)pda::max_tail_slots(n_cu, true));
}
"""


def test_batches_fit_the_chip_and_the_workspace(tmp_path):
    if not os.path.exists(CLANG):
        pytest.skip("no ROCm clang++ here")
    src, exe = tmp_path / "batch.cpp", tmp_path / "batch"
    src.write_text(MAIN)
    subprocess.run([CLANG, "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I", CSRC, str(src), "-o", str(exe)],
                   check=True, timeout=120)
    rng = random.Random(7)
    cases = [(1, 2048, 2048, 256, 24), (1, 2048, 0, 256, 24), (1, 9600, 9600, 256, 24), (2, 300, 390, 256, 7), (1, 2048, 2048, 256, 1)]
    for _ in range(3000):
        cases.append((rng.randint(1, 6), rng.randint(1, 12000), rng.choice([rng.randint(0, 700), rng.randint(1, 40000)]),
                      rng.choice([256, 256, 304, 64, 1]), rng.randint(1, 24)))
    out = subprocess.run([str(exe)], input="\n".join(" ".join(map(str, c)) for c in cases), capture_output=True, text=True, check=True, timeout=120)
    rows = [tuple(map(int, l.split())) for l in out.stdout.splitlines()]
    assert [k for k, _ in rows[:5]] == [8, 1, 1, 7, 1]
    for (BH, Sq, n_v, n_cu, left), (k, ws) in zip(cases, rows):
        plan = tail_plan(BH, Sq, n_v, 128, n_cu)
        items = plan["n_tiles"] + plan["n_cut"] * (plan["split"] - 1)
        assert 1 <= k <= max(left, 1)
        if k > 1:
            assert 2 * items <= n_cu and k * 2 * items <= 2 * n_cu            # every half item has its workgroup at once
            assert k * plan["workspace_slots"] <= ws
        elif left > 1 and n_v > 0:
            assert 2 * items > n_cu


@pytest.mark.gpu
@pytest.mark.parametrize("B,S,n_v,d,groups", [
    (1, 2100, 2100, 128, [1] * 11),                # cut in four: batches of seven and four
    (1, 2100, 2050, 64, [1] * 6),
    (2, 1300, 1300, 128, [2, 2, 2, 1]),            # two batches and heads, equal groups and one other
    (1, 300, 257, 128, [3, 3, 2, 2, 2]),           # nothing cut
    (1, 9600, 9600, 64, [1, 1]),                   # each group fills the chip: no batch
])
def test_groups_that_share_a_launch(B, S, n_v, d, groups):
    import torch
    import paper_2511_12056_amd as pda
    H = sum(groups)
    gen = torch.Generator(device="cuda").manual_seed(S + d)
    q, k, v = (torch.randn(B, H, S, d, generator=gen, device="cuda").to(torch.bfloat16) for _ in range(3))
    scale = d ** -0.5
    ref = torch.empty(B, H, S, d, device="cuda")
    rlse = torch.empty(B, H, S, device="cuda")
    h0 = 0
    for g in groups:
        sl = slice(h0, h0 + g)
        pda.attn_fwd_strided(q[:, sl], k[:, sl], v[:, sl], ref[:, sl], rlse[:, sl], scale, n_v)
        h0 += g
    torch.cuda.synchronize()
    cs, ds = torch.cuda.Stream(), torch.cuda.Stream()
    for layout in (pda.PDA_SINK_HEAD_MAJOR, pda.PDA_SINK_TOKEN_FINAL, pda.PDA_SINK_TOKEN_ARRIVAL):
        head_major = layout == pda.PDA_SINK_HEAD_MAJOR
        want = ref if head_major else ref.transpose(1, 2)
        ranks = 1 if head_major or H % 2 else 2
        if layout == pda.PDA_SINK_TOKEN_ARRIVAL:
            n, h = ranks, H // ranks                 # head i*h + j arrives in slot j*n + i
            want = want.reshape(B, S, n, h, d).transpose(2, 3).reshape(B, S, H, d)
        for timed in (False, True):
            out, lse = torch.full_like(ref, float("nan")), torch.full_like(rlse, float("nan"))
            sink = torch.full((B, H, S, d) if head_major else (B, S, H, d), float("nan"), device="cuda")
            torch.cuda.synchronize()
            times = pda.headchunk_run_ex(q, k, v, out, lse, scale, groups, cs, ds, sp_ranks=ranks, sink_layout=layout,
                                         kv_valid_len=n_v, sink=sink, timed=timed)
            cs.synchronize(); ds.synchronize()
            assert torch.equal(out, ref) and torch.equal(lse, rlse) and torch.equal(sink, want), (layout, timed)
            if timed:
                assert len(times[0]) == len(groups) and all(t > 0 for t in times[0])
