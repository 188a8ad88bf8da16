"""Second-order weights on long cells, up to 1100 times longer than wide in
either direction, where the squares beside the singular point take pieces that
grow with the distance (sides longer than 32/3 of it), against the oracle's
adaptive quadrature: fields of random densities, 1e-5 relative RMS of the vector
field per fluid, the bar of the second-order fields; and single weights and
their h derivatives read from a unit source, 2e-6 of the largest."""
import numpy as np
import pytest

import oracle as O

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nr,nphi,ratio,h", [(128, 4, 1.2, 0.1), (128, 16, 1.2, 0.018), (32, 16, 1.5, 0.05), (33, 16, 4.0, 0.05), (57, 4, 1.5, 0.05), (5, 256, 40.0, 0.05),
                                             (4, 512, 1e4, 0.05), (8, 128, 25.0, 0.05), (8, 256, 2.0, 0.05)])
def test_long_cells(nr, nphi, ratio, h):
    import paper_2506_10812_amd as sg
    from paper_2506_10812_amd import torch_ops as T
    aspect = 2 * np.pi / nphi / (np.log(ratio) / nr)
    print(f"hat aspect {nr}x{nphi} ratio {ratio}: cells {max(aspect, 1 / aspect):.0f} to 1", flush=True)
    rng = np.random.default_rng(nr + nphi)
    lo, hi = 0.7, 0.7 * ratio
    semi = nr & (nr - 1) != 0  # the semi-spectral operators
    sig = rng.uniform(0.5, 1.5, (1, nr, nphi)).astype(np.float32)
    at = np.arange(0, nr * nphi, max(1, nr * nphi // 257), dtype=np.int32)
    r = lo * np.exp((np.arange(nr) + 0.5) * np.log(ratio) / nr)
    if semi:
        S = T.SemiSpectral(nr, nphi, lo, hi, 1, sg.SECOND_ORDER)
        S.sigma.copy_(torch.tensor(sig))
        S.refresh(h * r[None])
        S.run()
        got = S.g_r, S.g_phi
        want = O.field_ring_hat(nr, nphi, lo, hi, h * r[None], sig.astype(np.float64), targets=at)
    else:
        F = T.FFTField([dict(n_r=nr, n_phi=nphi, r_min=lo, r_max=hi, h=[h])], sg.SECOND_ORDER)
        F.set_sigma(0, sig)
        F.run()
        got = F.g_r[0], F.g_phi[0]
        want = O.field_table(nr, nphi, lo, hi, [h], sig.astype(np.float64), targets=at, flags=O.SECOND_ORDER)
    got = np.stack([x.double().cpu().numpy().reshape(-1)[at] for x in got])
    want = np.stack([np.asarray(w).reshape(-1) for w in want])
    err = np.sqrt(((got - want) ** 2).sum() / (want ** 2).sum())
    print(f"  {err:.2e}", flush=True)
    assert err < 1e-5


@pytest.mark.parametrize("nr,nphi,ratio", [(64, 4, 1.2), (4, 512, 1e4)])
def test_weights_beside_the_singular_point(nr, nphi, ratio):
    import paper_2506_10812_amd as sg
    from paper_2506_10812_amd import torch_ops as T
    print(f"hat aspect weights {nr}x{nphi}", flush=True)
    lo, h = 0.7, 0.05
    du, dphi = np.log(ratio) / nr, 2 * np.pi / nphi
    F = T.FFTField([dict(n_r=nr, n_phi=nphi, r_min=lo, r_max=lo * ratio, h=[h])], sg.SECOND_ORDER)
    sig = np.zeros((1, nr, nphi), np.float32)
    i0, j0 = nr // 2, 1
    sig[0, i0, j0] = 1.0
    F.set_sigma(0, sig)
    F.run()
    gr, gp = (x[0, 0].double().cpu().numpy() / (-du * dphi) for x in (F.g_r[0][None], F.g_phi[0][None]))
    got, want = [], []
    for P in range(-2, 2):
        for Q in (-1, 0, 1, 2):
            w = O.hat_weight(P, Q, du, dphi, h, h)
            got.append((gr[i0 + P, (j0 + Q) % nphi], gp[i0 + P, (j0 + Q) % nphi]))
            want.append(w[:2])
    got, want = np.array(got), np.array(want, dtype=float)
    err = np.abs(got - want).max() / np.abs(want).max()
    print(f"  {err:.2e}", flush=True)
    assert err < 2e-6
