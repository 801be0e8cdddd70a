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


def _kernels(obj, name):
    """{symbol: [(mnemonic, operands)]} of the functions of a code object whose name contains `name`."""
    text = subprocess.run([os.path.join(LLVM, "llvm-objdump"), "-d", "--no-show-raw-insn", "--no-leading-addr", str(obj)],
                          check=True, capture_output=True, text=True, timeout=300).stdout
    out, code = {}, None
    for line in text.splitlines():
        head = re.match(r"(?:[0-9a-f]+ )?<(\w+)>:$", line)
        if head:
            code = out.setdefault(head[1], []) if name in head[1] else None
        elif code is not None:
            op, _, rest = line.split("//")[0].strip().partition(" ")
            if re.fullmatch(r"[a-z_0-9]+", op):
                code.append((op, rest.strip()))
    return out


def _waits_at_sweep_start(code, stores):
    """The vmcnt values waited for from the branch or memory access before it up to the wait for all but `stores`
    operations that is followed by the lane swaps of the Q fragments: the start of a sweep."""
    found = []
    for i, (op, args) in enumerate(code):
        if op != "s_waitcnt" or f"vmcnt({stores})" not in args or not any(o.startswith("v_permlane16_swap") for o, _ in code[i:i + 8]):
            continue
        waits = []
        for o, a in reversed(code[:i + 1]):
            if o.startswith(("s_cbranch", "s_branch", "buffer_", "global_", "scratch_", "flat_")):
                break
            m = re.search(r"vmcnt\((\d+)\)", a) if o == "s_waitcnt" else None
            if m:
                waits.append(int(m[1]))
        found.append(waits[::-1])
    return found


def test_next_sweep_does_not_wait_for_the_stores_before_it(code_objects):
    """An item's Q and first tiles are requested before the results of the item ahead of it are stored, and the
    sweep waits for all but those stores.  The compiler's own waits on the registers of Q, which it puts in front
    of that one, count the stores on the path with the fewest and must not ask for more."""
    kernels = {}
    for obj in code_objects:
        kernels.update(_kernels(obj, "attn_fwd_sp_kernel"))
    assert len(kernels) == 12
    for name, code in kernels.items():
        d, bf16 = re.search(r"attn_fwd_sp_kernelILi(\d+)ELi\dELb\dELb(\d)E", name).groups()
        stores = (2 if bf16 == "1" else 4) * int(d) // 32 + 1          # 64 bytes of 16 rows each, and the lse
        starts = _waits_at_sweep_start(code, stores)
        assert starts and all(min(w) >= stores for w in starts), (name, stores, starts)
