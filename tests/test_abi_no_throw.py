"""A host allocation that fails inside a call returns SG_ERR_HIP: no exception
crosses the C ABI.  In a process of its own, whose operator new (a small library
loaded ahead of libsg.so) throws when told to; the calls fail before they reach
the device, so their device pointers are made up."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

NEW = r"""
#include <cstdlib>
#include <new>
static int left = 0;
extern "C" void arm(int n) { left = n; }
extern "C" int armed() { return left; }
void *operator new(std::size_t n)
{
    if (left && --left == 0) throw std::bad_alloc();
    void *p = std::malloc(n ? n : 1);
    if (!p) throw std::bad_alloc();
    return p;
}
void operator delete(void *p) noexcept { std::free(p); }
void operator delete(void *p, std::size_t) noexcept { std::free(p); }
"""

SCRIPT = r"""
import ctypes, sys
shim = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
sys.path.insert(0, sys.argv[2])
import paper_2506_10812_amd as sg
L, g, f = sg.lib(), sg.grid(16, 32, 0.4, 2.5), sg.fluids([0.05])
P = 1 << 20
disc = (sg.Disc * 2)(*[sg.make_disc(g, f, 0, P, P, P, P)] * 2)
ms = (ctypes.c_float * 3)()
ref = ctypes.byref
calls = {
    "kernel_table": lambda: L.sg_kernel_table(ref(g), ref(f), 0, P, P, 1 << 40, 0),
    "field_fft 1": lambda: L.sg_field_fft(disc, 1, P, 1 << 40, 0),
    "field_fft 2": lambda: L.sg_field_fft(disc, 2, P, 1 << 40, 0),
    "profile": lambda: L.sg_field_fft_profile(disc, 1, P, 1 << 40, 0, 1, ms),
    "tune": lambda: L.sg_field_fft_tune(disc, 2, P, 1 << 40, 0, None, 0, None),
}
call = calls[sys.argv[3]]
shim.arm(1)
st = call()
assert shim.armed() == 0, "no allocation was made"
print("status", st, flush=True)
assert st == 3, st
"""


@pytest.mark.skipif(os.path.exists("/dev/kfd"), reason="made-up device pointers: only where no device can read them")
@pytest.mark.parametrize("call", ["kernel_table", "field_fft 1", "field_fft 2", "profile", "tune"])
def test_failed_allocation_returns_a_status(call, tmp_path):
    src, lib = tmp_path / "new.cpp", tmp_path / "libnew.so"
    src.write_text(NEW)
    subprocess.check_call(["g++", "-O1", "-shared", "-fPIC", str(src), "-o", str(lib)])
    r = subprocess.run([sys.executable, "-c", SCRIPT, str(lib), ROOT, call], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, (r.returncode, r.stdout, r.stderr[-800:])
