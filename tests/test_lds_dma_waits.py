"""Wait states in front of the global -> LDS loads of the built library.  The loads are written in inline
assembly, where the compiler's own insertion of wait states does not look, so the generated code is
checked: a load that takes its LDS address from M0 needs one wait state after a scalar write of M0, and
a vector memory instruction needs five after a VALU write (v_readlane of a spilled register, for
instance) of the scalar registers that hold its base."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2511_12056_amd", "libpipedit_attn.so")
OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"


def _sgprs(op):
    m = re.fullmatch(r"s\[(\d+):(\d+)\]", op)
    if m:
        return set(range(int(m[1]), int(m[2]) + 1))
    if op == "vcc":
        return {"vcc"}
    m = re.fullmatch(r"s(\d+)", op)
    return {int(m[1])} if m else ({"vcc"} if op in ("vcc_lo", "vcc_hi") else set())


def _sgprs_written_by_valu(op, args):
    """Scalar destinations of a vector ALU instruction (compares, readlanes, carries): among its first two operands."""
    if not op.startswith("v_"):
        return set()
    out = _sgprs(args[0]) if args else set()
    if len(args) > 1 and re.match(r"v_(add|sub|subrev|addc|subb|subbrev)_co_|v_mad_[iu]64|v_div_scale", op):
        out |= _sgprs(args[1])
    if op.startswith("v_cmp") and op.endswith("_e32"):
        out |= {"vcc"}
    return out


def violations(code):
    """code: list of (mnemonic, [operands]) in address order.  Walks back from each LDS load over the
    instructions before it in address order (a taken branch in between adds wait states of its own)."""
    bad = []
    loads = 0
    for i, (op, args) in enumerate(code):
        if not op.startswith("global_load_lds"):
            continue
        loads += 1
        base = _sgprs(args[1].split()[0])
        states = 0
        pending = set(base)                     # base registers whose writer has not been met yet
        for prev, pa in reversed(code[:i]):
            if states >= 5:
                break
            if states < 1 and prev.startswith("s_") and pa and pa[0] == "m0":
                bad.append((i, "m0 written by the instruction before"))
            if prev.startswith("s_") and pa:
                pending -= _sgprs(pa[0])        # a scalar write is interlocked
            if pending & _sgprs_written_by_valu(prev, pa):
                bad.append((i, f"base written by {prev} {states} states before"))
            states += int(pa[0], 0) + 1 if prev == "s_nop" else 1
    return loads, bad


def test_the_check_itself():
    ok = [("s_mov_b32", ["m0", "s0"]), ("s_mov_b64", ["vcc", "s[4:5]"]), ("global_load_lds_dwordx4", ["v1", "vcc"])]
    assert violations(ok) == (1, [])
    assert violations([("v_readlane_b32", ["s5", "v9", "3"])] + ok) == (1, [])          # copied by the scalar unit
    assert violations([("s_mov_b32", ["m0", "s0"]), ("global_load_lds_dwordx4", ["v1", "s[4:5]"])])[1]
    late = [("v_readlane_b32", ["s5", "v9", "3"]), ("s_mov_b32", ["m0", "s0"]), ("s_nop", ["2"]), ("global_load_lds_dwordx4", ["v1", "s[4:5]"])]
    assert violations(late)[1]
    late[2] = ("s_nop", ["3"])
    assert violations(late) == (1, [])


def test_every_lds_load_of_the_library_has_its_wait_states(tmp_path):
    if not (os.path.exists(OBJDUMP) and os.path.exists(LIB)):
        pytest.skip("no llvm-objdump or no built library here")
    lib = tmp_path / "lib.so"
    shutil.copy(LIB, lib)
    subprocess.run([OBJDUMP, "--offloading", str(lib)], cwd=tmp_path, check=True, capture_output=True, timeout=60)
    device = sorted(p for p in tmp_path.iterdir() if "gfx950" in p.name)
    assert device
    loads = 0
    for obj in device:
        text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", "--no-leading-addr", str(obj)],
                              check=True, capture_output=True, text=True, timeout=300).stdout
        code = []
        for line in text.splitlines():
            line = line.split("//")[0].strip()
            if not line or line.endswith(":") or not re.match(r"[a-z_0-9]+(\s|$)", line):
                continue
            op, _, rest = line.partition(" ")
            code.append((op, [a.strip() for a in rest.split(",")] if rest.strip() else []))
        n, bad = violations(code)
        loads += n
        assert not bad, (obj.name, len(bad), bad[:5])
    assert loads > 100                          # the attention kernels are in there
