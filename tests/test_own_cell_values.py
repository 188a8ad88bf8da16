"""Own-cell integrals of the oracle and of the library against values of 20
digits that share no code and no rule with either: mpmath Bessel functions at 32
digits, panels of ratio 3 towards the singular corner (the innermost graded as
t^4) times 30 nodes across.  Field (the X-symmetrised average of K_r over the
cell), its h_a and h_b derivatives, and the potential's average of P dA / (r^2 du
dphi) at r = 1, H = h.  Cells from 0.03 H to 15 H across a half side, either side
of 8 H, equal and unequal heights, aspects 1 to 500.

Bar: 1e-12 (the field's two halves cancel to about a half side, and so do the
digits of a double: 1e-16 over a half side of 1.5e-3 and sums of hundreds of
terms leave 1e-13)."""
import numpy as np
import pytest

import oracle as O

# n_r, n_phi, r_max / r_min, h_a, h_b: field, d/dh_a, d/dh_b, potential
VALUES = [
    (64, 128, 25, 0.05, 0.05, "-2.7566013098393520135",
     "73.912692775591600834", "-23.824578382233468248", "-24.886107184431896771"),
    (64, 128, 25, 0.05, 0.005, "-0.65740798519691024005",
     "25.088568531479738874", "-22.328041776859088153", "-30.010582937394566021"),
    (1024, 2048, 25, 0.05, 0.05, "-2.9363106757550449806",
     "86.422372874711177116", "-27.767261173375857111", "-55.719565994502601674"),
    (16, 64, 25, 0.0127, 0.0127, "-7.7297228697818830845",
     "187.3895940104303719", "-46.354008242613901803", "-20.344552958510603256"),
    (16, 64, 25, 0.0123, 0.03, "-7.8080896380164478457",
     "101.10577112201507455", "30.059010520584940595", "-18.072988017420457065"),
    (4, 64, 25, 0.05, 0.02, "-3.7074030537182458648",
     "30.525835127687953217", "-8.2575401150927091131", "-7.3793307386765433514"),
    (3, 2048, 100, 0.05, 0.05, "-3.5408840800582861295",
     "25.499475068301009994", "-0.086545054898890850105", "-5.256473126562578625"),
    (200, 8, 1.5, 0.05, 0.05, "2.5990737392271124873",
     "-11.625995692568796654", "-12.07659383731076612", "-7.7527176897034773128"),
]


@pytest.mark.parametrize("nr,nphi,ratio,ha,hb,field,da,db,pot", VALUES)
def test_oracle(nr, nphi, ratio, ha, hb, field, da, db, pot):
    du, dphi = np.log(ratio) / nr, 2 * np.pi / nphi
    for which, want in enumerate((field, da, db)):
        assert abs(O.self_cell(ha, hb, du, dphi, which) / float(want) - 1) < 1e-12, which
    for r in (1.0, 3.0):
        assert abs(O.potential_self(r, ha * r, hb * r, du, dphi) / (du * dphi * r * float(pot)) - 1) < 1e-12


@pytest.mark.gpu
@pytest.mark.parametrize("nr,nphi,ratio,ha,hb,field,da,db,pot", VALUES)
def test_library(nr, nphi, ratio, ha, hb, field, da, db, pot):
    torch = pytest.importorskip("torch")
    import paper_2506_10812_amd as sg
    from paper_2506_10812_amd import torch_ops as T
    print(f"own cell values {nr}x{nphi} h = {ha}, {hb}", flush=True)
    du, dphi = np.log(ratio) / nr, 2 * np.pi / nphi
    g = sg.grid(nr, nphi, 1.0, ratio)
    out = torch.empty(1, dtype=torch.float64, device="cuda")
    for which, want in enumerate((field, da, db)):
        sg.self_cell(g, [ha], [hb], which, out)
        err = abs(float(out[0]) / float(want) - 1)
        print(f"  which = {which}: {err:.1e}", flush=True)
        assert err < 1e-12
    # the potential of one cell's density at that cell, as the source's and as the target's fluid
    sig = torch.zeros((2, nr, nphi), dtype=torch.float64, device="cuda")
    sig[0, nr // 2, 1] = 1.0
    got = float(T.potential(g, [ha, hb], sig)[1, nr // 2, 1])
    err = abs(got / (du * dphi * np.exp((nr // 2 + 0.5) * du) * float(pot)) - 1)
    print(f"  potential: {err:.1e}", flush=True)
    assert err < 1e-12
