"""Own-cell integrals of the direct sums with one scale height per cell: every
rule of the quadrature (cell aspect ratio, cell side over H) and both launch
shapes (few cells, many cells with a cut-short last block), against the
oracle's own-cell quadrature.

The own-cell part is the difference of two sums, with and without it.
Tolerance: 1e-11 of the largest own-cell value (the bar of the own-cell
quadrature) plus the rounding of the two sums, 8 ulps of the largest value."""
import math

import numpy as np
import pytest

import oracle as O

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def sg():
    import paper_2506_10812_amd as m
    return m


@pytest.fixture(scope="module")
def T():
    from paper_2506_10812_amd import torch_ops as m
    return m


# (n_r, n_phi, fluids, aspect du/dphi): 63 x 67 cells leave 5 of 8 and 1 of 4
# cells in the last block; aspects on either side of each rule's limit (2, 8)
SHAPES = [(63, 67, 1, 1.0), (63, 67, 2, 1.9), (9, 13, 1, 2.1), (9, 13, 2, 0.2), (7, 10, 3, 0.11), (5, 9, 2, 9.0),
          (6, 7, 4, 0.6)]


@pytest.mark.parametrize("what", ["field", "potential"])
@pytest.mark.parametrize("nr,nphi,nf,aspect", SHAPES)
def test_own_cell_terms(sg, T, nr, nphi, nf, aspect, what):
    print(f"own cell {what} {nr}x{nphi} nf={nf} aspect={aspect}", flush=True)
    rng = np.random.default_rng(nr * nphi + nf)
    dphi = 2 * math.pi / nphi
    du = aspect * dphi
    rmin = 0.3
    rmax = rmin * math.exp(du * nr)
    r = rmin * np.exp((np.arange(nr) + 0.5) * du)
    half = 0.5 * max(du, dphi)
    # half side / H from 0.2 to 40: both radial rules, also within one block
    H = half / np.exp(rng.uniform(math.log(0.2), math.log(40.0), (nf, nr, nphi))) * r[None, :, None]
    H[:, : nr // 2] = half / rng.uniform(0.3, 7.5, (nf, nr // 2, nphi)) * r[None, : nr // 2, None]
    if nf > 1:
        H[1, 0] = H[0, 0]  # equal heights: the two sides of X = 0 share one evaluation
    sig = rng.uniform(0.5, 1.0, (nf, nr, nphi))
    g = sg.grid(nr, nphi, rmin, rmax)
    s, Ht = torch.tensor(sig, device="cuda"), torch.tensor(H, device="cuda")

    def call(flags):
        if what == "field":
            return T.direct(g, None, s, H=Ht, flags=flags)[0].cpu().numpy()
        return T.potential(g, None, s, H=Ht, flags=flags).cpu().numpy()

    full, excl = call(0), call(sg.SELF_CELL_EXCLUDE)
    own = full - excl
    cells = {(0, 0), (nr - 1, nphi - 1)} | {(int(rng.integers(nr)), int(rng.integers(nphi))) for _ in range(14)}
    got, want = [], []
    for i, j in sorted(cells):
        for b in range(nf):
            t = 0.0
            for a in range(nf):
                if what == "field":
                    k = float(O.self_cell(H[a, i, j] / r[i], H[b, i, j] / r[i], du, dphi))
                    t -= du * dphi * sig[a, i, j] * k
                else:
                    t += sig[a, i, j] * float(O.potential_self(r[i], H[a, i, j], H[b, i, j], du, dphi))
            want.append(t)
            got.append(own[b, i, j])
    got, want = np.array(got), np.array(want)
    tol = 1e-11 * np.abs(want).max() + 8 * np.finfo(float).eps * np.abs(full).max()
    err = np.abs(got - want).max()
    print(f"  err {err:.2e} tol {tol:.2e}", flush=True)
    assert err < tol
