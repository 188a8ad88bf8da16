"""The tables that the kernels read (csrc/gen_cheb64.cpp, written at build time)
on the CPU: the local polynomials of F, D = -x F' - 3/2 F, G0 = e^x K0 and E =
2 x F - G0, those of V(u) = u^{-3/2} F(1/u) and Vg(u) = u^{-1/2} G0(1/u) in double
and in float, and the double twiddles.

The polynomials are summed in long double with the device's interval and local
variable (the leading mantissa bits choose the interval, the rest is v in [1, 1 +
1/n), t = 2 n v - 2 n - 1) at both ends of every interval and a point between, against
30-digit values; so what is left is the rounding of the coefficients,
half a unit of each (together 1.3 times the leading one) and the truncation:
2.5e-16 in double, 1.2e-7 in float."""
import os
import re
import subprocess

import numpy as np
import pytest

mp = pytest.importorskip("mpmath")

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
GEN = os.path.join(ROOT, "paper_2506_10812_amd", "csrc", "gen_cheb64.cpp")


@pytest.fixture(scope="module")
def header(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("tables") / "gen")
    subprocess.check_call(["g++", "-O2", "-std=c++17", GEN, "-o", exe])
    out = subprocess.run([exe, "--header"], capture_output=True, text=True, check=True).stdout
    const = {k: int(v) for k, v in re.findall(r"#define (\w+) (-?\d+)", out)}
    arrays = {k: np.array([float(x.rstrip("f")) for x in v.replace(",", " ").split()],  # float: as the compiler reads it
                          dtype=np.float32 if k == "sg_polyu32" else np.float64)
              for k, v in re.findall(r"const (?:double|float) (\w+)\[[^]]*\] = \{\n(.*?)\};", out, re.S)}
    return const, arrays


def _value(fn, x):
    k0, k1 = mp.besselk(0, x), mp.besselk(1, x)
    if fn in ("G0", "Vg"):
        return mp.exp(x) * k0
    F = mp.exp(x) * (k1 - k0)
    if fn in ("F", "V"):
        return F
    dF = mp.exp(x) * (2 * (k1 - k0) - k1 / x)
    return -x * dF - 1.5 * F if fn == "D" else 2 * x * F - mp.exp(x) * k0


CASES = [("sg_poly64", 0, "F"), ("sg_poly64", 1, "D"), ("sg_poly64", 2, "G0"), ("sg_poly64", 3, "E"),
         ("sg_polyu64", 0, "V"), ("sg_polyu64", 1, "Vg"), ("sg_polyu32", 0, "V"), ("sg_polyu32", 1, "Vg")]


@pytest.mark.parametrize("table,row,fn", CASES)
def test_local_polynomials(header, table, row, fn):
    const, arrays = header
    mp.mp.dps = 32
    single = table == "sg_polyu32"
    sub = const["SG_POLYF_SUB" if single else "SG_POLY_SUB"]
    oct0 = const["SG_POLYF_OCT0" if single else "SG_POLYU_OCT0" if table == "sg_polyu64" else "SG_POLY_OCT0"]
    ni, nc = (const["SG_POLYF_NI"], const["SG_POLYF_NC"]) if single else (const["SG_POLY_NI"], const["SG_POLY_NC"])
    c = arrays[table].reshape(-1, ni, nc + 1 if single else nc)[row]
    if single:
        assert np.all(c[:, nc] == 0)  # padding of the 16-byte reads
    worst = 0.0
    for k in range(ni):
        lo = 2.0 ** (oct0 + k // sub) * (1 + (k % sub) / sub)
        width = 2.0 ** (oct0 + k // sub) / sub
        for x in (lo, lo + 0.37 * width, np.nextafter(lo + width, 0)):
            m, e = np.frexp(x)
            assert int((2 * m - 1) * sub) + sub * (int(e) - 1 - oct0) == k
            v = 2 * m - (k % sub) / sub
            t = np.longdouble(2 * sub) * np.longdouble(v) - (2 * sub + 1)
            assert -1 <= t < 1
            got = np.longdouble(0)
            for a in c[k, nc - 1::-1]:
                got = got * t + np.longdouble(a)
            if fn in ("V", "Vg"):
                w = _value(fn, 1 / mp.mpf(x)) * mp.mpf(x) ** (mp.mpf(-3) / 2 if fn == "V" else mp.mpf(-1) / 2)
            else:
                w = _value(fn, mp.mpf(x))
            # relative to the interval's value (E changes sign: to its largest there)
            scale = max(abs(w), mp.mpf(float(abs(c[k, 0]))))
            worst = max(worst, float(abs(mp.mpf(str(got)) - w) / scale))
    print(f"{table} {fn}: {worst:.2e}")
    assert worst < (1.2e-7 if single else 2.5e-16)


def test_twiddles(header):
    const, arrays = header
    n = const["SG_TW64_N"]
    tw = arrays["sg_tw64"].reshape(n, 2)
    mp.mp.dps = 30
    for k in range(0, n, 1):
        a = 2 * mp.pi * k / n
        assert abs(tw[k, 0] - mp.cos(a)) < 1.2e-16 and abs(tw[k, 1] - mp.sin(a)) < 1.2e-16, k


def test_header_holds_nothing_else(header):
    assert set(header[1]) == {"sg_poly64", "sg_polyu64", "sg_polyu32", "sg_tw64"}
