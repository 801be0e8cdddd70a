"""The rule that picks the workgroup size of an attention launch (host code of the kernel's header,
compiled here on its own) against the same rule written out in Python, which the GPU tests use to say
which kernel they reach."""
import os
import random
import subprocess

import pytest

from tests.util import wavefronts

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2511_12056_amd", "csrc")
CLANG = "/opt/rocm/llvm/bin/clang++"
MAIN = r"""
#include "attn_internal.h"
#include <stdio.h>
int main() {
    long long Sq, n_v;
    int BH, d, n_cu;
    while (scanf("%d %lld %lld %d %d", &BH, &Sq, &n_v, &d, &n_cu) == 5)
        printf("%d\n", pda::sp_wavefronts(pda::plan_tail(Sq, BH, n_v, n_cu), n_v, d, n_cu));
}
"""


def test_workgroup_size_rule(tmp_path):
    if not os.path.exists(CLANG):
        pytest.skip("no ROCm clang++ here")
    src, exe = tmp_path / "rule.cpp", tmp_path / "rule"
    src.write_text(MAIN)
    subprocess.run([CLANG, "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I", CSRC, str(src), "-o", str(exe)],
                   check=True, timeout=120)
    rng = random.Random(64)
    cases = [(1, 300, 700, 128, 256), (200, 300, 700, 128, 256), (193, 1900, 1, 128, 256), (130, 1900, 192, 128, 256),
             (130, 1900, 256, 128, 256), (130, 1900, 448, 64, 256), (130, 1900, 449, 64, 256), (128, 2000, 700, 128, 256),
             (160, 2000, 700, 64, 256), (24, 16384, 1536, 128, 256), (24, 16384, 1537, 128, 256)]
    for n_cu in (256, 256, 256, 304, 64, 1):
        for _ in range(1500):
            tph = rng.choice([1, 2, 3, 4, 7, 8, 9, rng.randint(1, 500)])
            BH = max(1, round(n_cu * rng.choice([0.1, 0.5, 1, 4, 4.06, 4.5, 4.6, 5, 5.5, 6, 9, rng.uniform(0, 12)]) / tph))
            n_v = max(1, rng.choice([rng.randint(1, 2000), 64 * rng.randint(1, 30), rng.randint(1, 120000)]))
            cases.append((BH, tph * 256 - rng.randint(0, 255), n_v, rng.choice([64, 128]), n_cu))
    out = subprocess.run([str(exe)], input="\n".join(" ".join(map(str, c)) for c in cases), capture_output=True, text=True, check=True, timeout=120)
    got = [int(x) for x in out.stdout.split()]
    assert got == [wavefronts(*c) for c in cases]
    assert got[:11] == [4, 8, 4, 8, 4, 8, 4, 8, 8, 4, 8] and 0.1 < got.count(4) / len(got) < 0.9
