"""Which base-2 launches at d = 64 start with pairs of tiles: the rule against the same rule written out here, on both
sides of each of its lines."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2511_12056_amd", "csrc")
CLANG = "/opt/rocm/llvm/bin/clang++"
MAIN = r"""
#include "attn_internal.h"
#include <stdio.h>
int main() {
    long long Sq, n_v;
    int BH, d, base2;
    while (scanf("%d %lld %lld %d %d", &BH, &Sq, &n_v, &d, &base2) == 5)
        printf("%d\n", (int)pda::wide_pays(pda::plan_tail(Sq, BH, n_v, 256), n_v, d, base2 != 0, 256));
}
"""


def test_rule(tmp_path):
    if not os.path.exists(CLANG):
        pytest.skip("no ROCm clang++ here")
    src, exe = tmp_path / "pays.cpp", tmp_path / "pays"
    src.write_text(MAIN)
    subprocess.run([CLANG, "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I", CSRC, str(src), "-o", str(exe)],
                   check=True, timeout=120)
    lines = {511: 9600, 512: 3072, 1024: 3072, 1025: 768}        # tiles of the launch: most keys with pairs
    cases = [(tiles, 256, n_v, d, base2) for tiles in lines for n_v in (224, 768, 769, 3072, 3073, 9600, 9601, 119056)
             for d in (64, 128) for base2 in (0, 1)]
    out = subprocess.run([str(exe)], input="\n".join(" ".join(map(str, c)) for c in cases), capture_output=True, text=True, check=True, timeout=120)
    assert [int(l) for l in out.stdout.split()] == [int(d != 64 or not base2 or n_v <= lines[tiles]) for tiles, _, n_v, d, base2 in cases]
