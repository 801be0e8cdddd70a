"""Resources of the kernels of the built library, from its code objects."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2511_12056_amd", "libpipedit_attn.so")
LLVM = "/opt/rocm/llvm/bin"


@pytest.fixture(scope="module")
def code_objects(tmp_path_factory):
    if not (os.path.exists(os.path.join(LLVM, "llvm-objdump")) and os.path.exists(LIB)):
        pytest.skip("no llvm-objdump or no built library here")
    tmp = tmp_path_factory.mktemp("code")
    lib = tmp / "lib.so"
    shutil.copy(LIB, lib)
    subprocess.run([os.path.join(LLVM, "llvm-objdump"), "--offloading", str(lib)], cwd=tmp, check=True, capture_output=True, timeout=60)
    found = sorted(p for p in tmp.iterdir() if "gfx950" in p.name)
    assert found
    return found


def test_no_kernel_needs_scratch_memory(code_objects):
    """A kernel with a private segment makes the runtime provide scratch memory for the queue it runs on, which
    the attention entry points, and pda_attn_fwd_noalloc above all, do not ask for."""
    sizes = {}
    for obj in code_objects:
        notes = subprocess.run([os.path.join(LLVM, "llvm-readelf"), "--notes", str(obj)], check=True, capture_output=True,
                               text=True, timeout=60).stdout
        names = re.findall(r"^ +\.name: +(_Z\w+)$", notes, re.M)
        private = re.findall(r"^ +\.private_segment_fixed_size: +(\d+)$", notes, re.M)
        assert len(names) == len(private)
        sizes.update(zip(names, map(int, private)))
    assert sum("attn_fwd_sp_kernel" in n for n in sizes) == 12
    assert {n: b for n, b in sizes.items() if b} == {}
