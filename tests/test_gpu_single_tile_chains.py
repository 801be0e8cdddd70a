"""Rows that need the second sweep in chains of single tiles: items that sweep a second time, for one row of a wavefront or
for all rows, between items that do not, in launches without pairs of tiles and with more than one item per workgroup."""
import math
import os
import random
import subprocess

import numpy as np
import pytest

from synth import bf16_bits_to_f32, f32_to_bf16_bits
from tests.test_gpu_launch_forms import _launch, _repeat
from tests.test_gpu_rows_form import rows_form
from tests.test_gpu_wide_items import wide_plan
from tests.util import LSE_REL, REL_L2, cut_row_mask, tail_plan, to_dev_bf16, wavefronts

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2511_12056_amd", "csrc")
CLANG = "/opt/rocm/llvm/bin/clang++"
MAIN = r"""
#include "attn_internal.h"
#include <stdio.h>
int main() {
    long long Sq, n_v;
    int BH, d, base2, n_cu;
    while (scanf("%d %lld %lld %d %d %d", &BH, &Sq, &n_v, &d, &base2, &n_cu) == 6) {
        const auto t = pda::plan_tail(Sq, BH, n_v, n_cu);
        const bool rows = pda::rows_form(t, Sq, BH, n_v, d, n_cu);
        const bool wide = !rows && pda::wide_pays(t, n_v, d, base2 != 0, n_cu) && pda::wide_plan(t, n_v, n_cu).items > 0;
        printf("%d\n", rows ? 1 : wide ? 2 : pda::sp_wavefronts(t, n_v, d, n_cu));
    }
}
"""


def kernel(BH, Sq, n_v, d, base2, n_cu):
    """What a launch of one group takes: "rows" (few query rows), "pairs" (pairs of tiles first), or single tiles in workgroups of
    4 or 8 wavefronts."""
    if rows_form(BH, Sq, n_v, d, n_cu):
        return "rows"
    tiles = tail_plan(BH, Sq, n_v, d, n_cu)["n_tiles"]
    most = math.inf if d == 128 or not base2 else 9600 if tiles < 2 * n_cu else 3072 if tiles <= 4 * n_cu else 768
    if n_v <= most and wide_plan(BH, Sq, n_v, n_cu)[0]:
        return "pairs"
    return wavefronts(BH, Sq, n_v, d, n_cu)


def test_rule(tmp_path):
    if not os.path.exists(CLANG):
        pytest.skip("no ROCm clang++ here")
    src, exe = tmp_path / "kernel.cpp", tmp_path / "kernel"
    src.write_text(MAIN)
    subprocess.run([CLANG, "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I", CSRC, str(src), "-o", str(exe)],
                   check=True, timeout=120)
    rng = random.Random(8)
    cases = []
    for n_cu in (256, 256, 304):
        for _ in range(1200):
            tph = rng.choice([1, 2, 3, 8, rng.randint(1, 100)])
            BH = max(1, round(n_cu * rng.choice([0.05, 0.3, 1, 2, 4, 4.1, 6, rng.uniform(0, 8)]) / tph))
            cases.append((BH, tph * 256 - rng.randint(0, 255), rng.choice([rng.randint(1, 2000), rng.randint(1, 20000)]), rng.choice([64, 128]),
                          rng.randint(0, 1), n_cu))
    out = subprocess.run([str(exe)], input="\n".join(" ".join(map(str, c)) for c in cases), capture_output=True, text=True, check=True, timeout=120)
    got = [{1: "rows", 2: "pairs"}.get(int(x), int(x)) for x in out.stdout.split()]
    assert got == [kernel(*c) for c in cases]
    assert all(got.count(x) > 100 for x in ("rows", "pairs", 4, 8))


@pytest.mark.gpu
@pytest.mark.parametrize("H,Sq,n_v,d,entry,form", [
    (193, 1900, 190, 128, "fp32", 4), (193, 1900, 190, 128, "bf16", 4), (193, 1900, 190, 128, "base2", 4),      # too few keys for pairs
    (130, 2000, 180, 64, "fp32", 8), (130, 2000, 180, 64, "bf16", 8), (130, 2000, 180, 64, "base2", 8),
    (600, 250, 700, 128, "fp32", 8), (600, 250, 700, 128, "bf16", 8), (600, 250, 700, 128, "base2", 8),        # one tile per head
    (600, 250, 700, 64, "fp32", 8), (600, 250, 700, 64, "bf16", 8),
    (193, 1900, 769, 64, "base2", 4), (193, 1900, 1536, 64, "base2", 4),                                      # base 2, d = 64: pairs do not pay
    (130, 2000, 1700, 64, "base2", 8),
    (193, 1900, 768, 64, "base2", "pairs"),                                                                   # ... and where they do
])
def test_second_sweep_between_other_items(H, Sq, n_v, d, entry, form):
    """The item after one that sweeps twice, and the rows beside such a row: heads of the same content, which different items
    precede, have the same bits, and those of the oracle to rounding."""
    import torch
    from oracle import attention
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    if n_cu == 256:
        assert kernel(H, Sq, n_v, d, entry == "base2", 256) == form
        plan = tail_plan(H, Sq, n_v, d, 256)
        assert plan["n_tiles"] > 256 and (plan["n_cut"] == 0 or entry == "base2")
    base = 5
    row_a, row_b = Sq - 3, 100                                    # the last wavefront of a tile, and one in the middle
    rng = np.random.default_rng(n_v + d)
    q = rng.standard_normal((1, base, Sq, d)).astype(np.float32)
    k = (rng.standard_normal((1, base, n_v, d)) * 0.05).astype(np.float32)
    v = rng.standard_normal((1, base, n_v, d)).astype(np.float32)
    k[0, 1, n_v - 20] = q[0, 1, row_a] * np.float32(1.5 * 128 / d)        # > 64 log2 units above the first tile
    k[0, 1, n_v - 50] = q[0, 1, row_b] * np.float32(1.5 * 128 / d)
    k[0, 2, n_v - 70] = q[0, 2, row_b] * np.float32(0.45 * 128 / d)       # ~50 log2 units, times values of 2^90
    v[0, 2] *= np.float32(2.0 ** 90)
    k[0, 4, 100:] *= np.float32(600.0)                                    # every row, every tile
    qb, kb, vb = (f32_to_bf16_bits(x) for x in (q, k, v))
    oracle_scale = 1.0
    if entry == "base2":
        qb, oracle_scale = f32_to_bf16_bits(q * np.float32(math.log2(math.e))), math.log(2.0)
    for row in (row_a, row_b):
        s = bf16_bits_to_f32(kb[0, 1]).astype(np.float64) @ bf16_bits_to_f32(qb[0, 1, row]).astype(np.float64) * oracle_scale
        assert s[64:].max() - s[:64].max() > 64 * math.log(2.0)
    dq, dk, dv = to_dev_bf16(qb), to_dev_bf16(kb), to_dev_bf16(vb)
    out, lse = _launch(entry, _repeat(dq, H), _repeat(dk, H), _repeat(dv, H), 1.0)
    ro, rl = attention(qb, kb, vb, oracle_scale)
    whole = torch.ones(H, Sq, dtype=torch.bool, device="cuda")
    if tail_plan(H, Sq, n_v, d, n_cu)["n_cut"]:
        whole = torch.from_numpy(~cut_row_mask(1, H, Sq, n_v, d, n_cu)[0]).cuda()
    first = {}
    for h in range(H):
        o, l, w = first.setdefault(h % base, (out[0, h], lse[0, h], whole[h]))
        both = w & whole[h]
        assert torch.equal(out[0, h][both], o[both]) and torch.equal(lse[0, h][both], l[both]), h
    tol = REL_L2 + (2.0 ** -9 / np.sqrt(3.0) if entry == "bf16" else 0.0)
    for h in [*range(base), *range(H - base, H)]:                 # relative gates: one head spans 2^90
        o, l = out[0, h].double().cpu().numpy(), lse[0, h].double().cpu().numpy()
        assert np.isfinite(o).all() and np.isfinite(l).all()
        assert np.sqrt(((o - ro[0, h % base]) ** 2).sum() / (ro[0, h % base] ** 2).sum()) <= tol, h
        assert (np.abs(l - rl[0, h % base]) / np.maximum(np.abs(rl[0, h % base]), 1.0)).max() <= LSE_REL, h
