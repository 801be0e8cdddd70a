"""Wait states in the generated code of the built library, where it holds inline assembly: the compiler's own insertion of
wait states does not look into it.

Global -> LDS loads: a load that takes its LDS address from M0 needs one wait state after a scalar write of M0, and
a vector memory instruction needs five after a VALU write (v_readlane of a spilled register, for
instance) of the scalar registers that hold its base.

MFMAs: a VALU write of a vector register needs two wait states before an MFMA that reads it as an operand."""
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


def _vgprs(op):
    m = re.fullmatch(r"([va])\[(\d+):(\d+)\]", op)
    if m:
        return {(m[1], i) for i in range(int(m[2]), int(m[3]) + 1)}
    m = re.fullmatch(r"([va])(\d+)", op)
    return {(m[1], int(m[2]))} if m else set()


def mfma_violations(code):
    """Walks back from each MFMA over the two wait states before it: VALU writes of its operands."""
    bad = []
    mfmas = 0
    for i, (op, args) in enumerate(code):
        if not op.startswith("v_mfma"):
            continue
        mfmas += 1
        operands = set().union(*map(_vgprs, args[1:4]))
        states = 0
        for prev, pa in reversed(code[:i]):
            if states >= 2:
                break
            if prev.startswith("v_") and not prev.startswith("v_mfma"):
                if operands & (_vgprs(pa[0]) | (_vgprs(pa[1]) if "swap" in prev else set())):
                    bad.append((i, f"operand written by {prev} {states} states before"))
            states += int(pa[0], 0) + 1 if prev == "s_nop" else 1
    return mfmas, bad


def test_the_mfma_check_itself():
    move, mfma = ("v_mov_b32_e32", ["v143", "v236"]), ("v_mfma_f32_32x32x16_bf16", ["v[128:143]", "v[224:227]", "v[160:163]", "v[128:143]"])
    assert mfma_violations([move, ("s_nop", ["1"]), mfma]) == (1, [])
    assert mfma_violations([move, ("s_nop", ["0"]), mfma])[1]
    assert mfma_violations([move, ("s_waitcnt", ["lgkmcnt(2)"]), mfma])[1]
    assert mfma_violations([move, ("s_nop", ["0"]), ("s_waitcnt", ["lgkmcnt(2)"]), mfma]) == (1, [])
    assert mfma_violations([("v_permlane32_swap_b32_e32", ["v1", "v160"]), mfma])[1]
    assert mfma_violations([("v_mov_b32_e32", ["v144", "v160"]), mfma]) == (1, [])


def _instructions(obj):
    text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", "--no-leading-addr", str(obj)],
                          check=True, capture_output=True, text=True, timeout=300).stdout
    code = []
    for line in text.splitlines():
        line = line.split("//")[0].strip()
        if not line or line.endswith(":") or not re.match(r"[a-z_0-9]+(\s|$)", line):
            continue
        op, _, rest = line.partition(" ")
        code.append((op, [a.strip() for a in rest.split(",")] if rest.strip() else []))
    return code


@pytest.fixture(scope="module")
def device_code(tmp_path_factory):
    """{code object: its instructions}"""
    if not (os.path.exists(OBJDUMP) and os.path.exists(LIB)):
        pytest.skip("no llvm-objdump or no built library here")
    tmp = tmp_path_factory.mktemp("code")
    lib = tmp / "lib.so"
    shutil.copy(LIB, lib)
    subprocess.run([OBJDUMP, "--offloading", str(lib)], cwd=tmp, check=True, capture_output=True, timeout=60)
    device = sorted(p for p in tmp.iterdir() if "gfx950" in p.name)
    assert device
    return {obj.name: _instructions(obj) for obj in device}


def test_every_lds_load_of_the_library_has_its_wait_states(device_code):
    loads = 0
    for name, code in device_code.items():
        n, bad = violations(code)
        loads += n
        assert not bad, (name, len(bad), bad[:5])
    assert loads > 100                          # the attention kernels are in there


def test_every_mfma_of_the_library_has_its_wait_states(device_code):
    mfmas = 0
    for name, code in device_code.items():
        n, bad = mfma_violations(code)
        mfmas += n
        assert not bad, (name, len(bad), bad[:5])
    assert mfmas > 1000
