"""No C++ exception leaves a C entry point: the pipeline calls, which build lists on the host, in a process whose
operator new fails.  The failure is switched on around each call only; nothing reaches a GPU."""
import os
import shutil
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
NEW = r"""
#include <cstdlib>
#include <new>
static bool failing = false;
extern "C" void fail_new(int on) { failing = on != 0; }
void* operator new(std::size_t n) {
    void* p = failing ? nullptr : std::malloc(n);
    if (!p) throw std::bad_alloc();
    return p;
}
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, std::size_t) noexcept { std::free(p); }
"""
CHILD = r"""
import ctypes as C, sys
new, lib = C.CDLL(sys.argv[1]), C.CDLL(sys.argv[2])
lib.pda_last_error.restype = C.c_char_p
p, n, i64, sizes = C.c_void_p(4096), None, C.c_int64(64), (C.c_int * 4)(1, 1, 1, 1)
a = [p, p, p, p, p, 1, 4, i64, i64, 64, C.c_float(0.125), i64]
for call in (lambda: lib.pda_headchunk_run(*a, 1, p, n, n, n, n),
             lambda: lib.pda_headchunk_run_ex(*a, sizes, 4, 1, 0, p, n, n, n, n)):
    new.fail_new(1)
    rc = call()
    new.fail_new(0)
    print(rc, lib.pda_last_error().decode(), flush=True)
"""


def test_failing_host_allocation(tmp_path):
    if not shutil.which("g++"):
        pytest.skip("no g++ here")
    from paper_2511_12056_amd import lib_path
    src, so = tmp_path / "new.cpp", tmp_path / "new.so"
    src.write_text(NEW)
    subprocess.run(["g++", "-O1", "-shared", "-fPIC", str(src), "-o", str(so)], check=True, timeout=60)
    preload = os.environ.get("LD_PRELOAD", "")
    env = dict(os.environ, LD_PRELOAD=str(so) + (":" + preload if preload else ""))
    res = subprocess.run([sys.executable, "-c", CHILD, str(so), lib_path()], cwd=ROOT, env=env, capture_output=True, text=True, timeout=120)
    assert res.returncode == 0, (res.returncode, res.stdout, res.stderr[-500:])
    lines = res.stdout.splitlines()
    assert len(lines) == 2 and all(l.startswith("4 no host memory") for l in lines), lines
