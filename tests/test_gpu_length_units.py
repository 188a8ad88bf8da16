"""The direct sums in other units of length: the field of a density depends on
lengths only through H/r, the potential is proportional to them.  Lengths
times a power of two change no digit of the inputs, so a float call in
centimetres (r of 10^15) gives the digits of one with r near 1 up to the
rounding of radii formed as exp(ln r_min + ...), 2^-52 ln r_min: one unit of
the last place at most.  From 10^-27 to 10^27."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
TOL = {"f32": 2.0 ** -22, "f64": 1e-13}


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("kind", ["rings", "cells", "rings LINEAR_R", "cells LINEAR_R", "cells INDIRECT", "potential rings",
                                  "potential cells"])
def test_units_of_length(kind, dtype):
    import paper_2506_10812_amd as sg
    from paper_2506_10812_amd import torch_ops as T
    print(f"length units {kind} {dtype}", flush=True)
    nr, nphi, nf = 17, 40, 2
    flags = sum(getattr(sg, k) for k in kind.split() if k.isupper())
    tt = torch.float32 if dtype == "f32" else torch.float64
    gen = torch.Generator().manual_seed(3)
    sig = (0.5 + torch.rand((nf, nr, nphi), generator=gen, dtype=torch.float64)).to(tt).cuda()
    H = (0.06 + 0.02 * torch.rand((nf, nr, nphi), generator=gen, dtype=torch.float64)).to(tt).cuda()

    def solve(k):
        L = 2.0 ** k
        g = sg.grid(nr, nphi, 1.5 * L, 18.0 * L)
        Hk = (H * L).contiguous() if "cells" in kind else None
        if "potential" in kind:
            return [T.potential(g, [0.05, 0.02], sig, Hk, flags).double() / L]
        return [x.double() for x in T.direct(g, [0.05, 0.02], sig, Hk, flags)]

    want = solve(0)
    for k in (-90, -43, 40, 43, 50, 90):
        for a, b in zip(solve(k), want):
            err = float((a - b).abs().max() / b.abs().max())
            print(f"  2^{k}: {err:.1e}", flush=True)
            assert err <= TOL[dtype]
