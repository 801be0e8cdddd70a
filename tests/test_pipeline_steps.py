"""The launches of a head-group pipeline (host code of the kernel's header, compiled here on its own): the same
ones as asking for every group anew, from a number of looks at the group list that grows with its length only."""
import os
import random
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2511_12056_amd", "csrc")
CLANG = "/opt/rocm/llvm/bin/clang++"
MAIN = r"""
#include "attn_internal.h"
#include <stdio.h>
struct Counted {
    std::vector<int> v;
    mutable long long looks = 0;
    size_t size() const { return v.size(); }
    int operator[](int i) const { ++looks; return v[i]; }
};
int main() {
    long long Sq, n_v;
    int B, n_cu, alone, n;
    while (scanf("%d %lld %lld %d %d %d", &B, &Sq, &n_v, &n_cu, &alone, &n) == 6) {
        Counted s;
        s.v.resize(n);
        for (int& x : s.v) if (scanf("%d", &x) != 1) return 1;
        const auto steps = pda::pipeline_steps(s, B, Sq, n_v, n_cu, alone != 0);
        bool same = true;
        size_t i = 0;
        for (int g = 0, h0 = 0; n <= 200 && g < n; ++i) {            // group by group, each time over all that remain
            int equal = 1;
            while (g + equal < n && s.v[g + equal] == s.v[g]) ++equal;
            const int k = alone ? 1 : pda::batch_of_groups(Sq, B * s.v[g], n_v, n_cu, equal);
            same = same && i < steps.size() && steps[i].h0 == h0 && steps[i].hg == s.v[g] && steps[i].groups == k;
            h0 += k * s.v[g];
            g += k;
        }
        printf("%d %lld %zu\n", n > 200 || (same && i == steps.size()), s.looks, steps.size());
    }
}
"""


def test_steps_of_a_pipeline(tmp_path):
    if not os.path.exists(CLANG):
        pytest.skip("no ROCm clang++ here")
    src, exe = tmp_path / "steps.cpp", tmp_path / "steps"
    src.write_text(MAIN)
    subprocess.run([CLANG, "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I", CSRC, str(src), "-o", str(exe)],
                   check=True, timeout=120)
    rng = random.Random(11)
    cases = [(1, 40000, 64, 256, 0, [1] * 65535), (1, 2048, 2048, 256, 0, [1] * 65535), (1, 2048, 2048, 256, 1, [1] * 65535),
             (1, 2048, 2048, 256, 0, [1] * 24), (1, 2048, 2048, 256, 0, [])]
    for _ in range(600):
        sizes = [x for _ in range(rng.randint(1, 5)) for x in [rng.randint(1, 4)] * rng.randint(1, 20)]
        cases.append((rng.randint(1, 3), rng.randint(1, 12000), rng.choice([0, rng.randint(1, 700), rng.randint(1, 40000)]),
                      rng.choice([256, 304, 64, 1]), rng.randint(0, 1), sizes))
    text = "\n".join(" ".join(map(str, (*c[:5], len(c[5]), *c[5]))) for c in cases)
    out = subprocess.run([str(exe)], input=text, capture_output=True, text=True, check=True, timeout=120)
    rows = [tuple(map(int, l.split())) for l in out.stdout.splitlines()]
    assert len(rows) == len(cases)
    for c, (same, looks, _) in zip(cases, rows):
        assert same and looks <= 3 * len(c[5]), (c[:5], len(c[5]), same, looks)
    assert [n for _, _, n in rows[:5]] == [65535, 8192, 65535, 3, 0]
