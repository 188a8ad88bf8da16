"""The functions behind the scale-height derivatives beyond x = 256, where they
take asymptotic series: D = -x F' - 3/2 F and, of the potential, E = 2 x F -
G0.  dL/dH of one ring pull on another (Sigma = 1 on ring i', lam_r = 1 on ring
i, both constant in phi, whose transforms are exact) is one sum of these
functions over four azimuths, nearly all of it from phi = 0, whose x is 257.
Against the series through n = 11 in double: about 20 roundings, 5e-15."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["field", "potential"])
@pytest.mark.parametrize("x_at", [257.0, 300.0, 1000.0])
def test_derivatives_beyond_the_polynomials(kind, x_at):
    import paper_2506_10812_amd as sg
    from paper_2506_10812_amd import torch_ops as T
    print(f"function tail {kind} x = {x_at}", flush=True)
    n_r, n_phi, k, h = 9, 4, 4, 0.005
    # x at phi = 0 of rings k apart: (cosh X - 1) / (4 h^2 cosh X)
    X = np.arccosh(1.0 / (1.0 - 4 * h * h * x_at))
    du = X / k
    lo = 1.5
    hi = lo * np.exp(n_r * du)
    du = np.log(hi / lo) / n_r
    X = k * du
    S = T.SemiSpectral(n_r, n_phi, lo, hi, 1, sg.POTENTIAL if kind == "potential" else 0)
    r = np.exp(np.log(lo) + (np.arange(n_r) + 0.5) * du)
    H = torch.tensor(h * r[None], device="cuda")
    S.refresh(H)
    ip, i = 2, 2 + k
    S.sigma.zero_()
    S.sigma[0, ip] = 1.0
    lam, zero = torch.zeros_like(S.sigma), torch.zeros_like(S.sigma)
    lam[0, i] = 1.0
    dH = torch.empty((1, n_r), dtype=torch.float64, device="cuda")
    ws = torch.empty(sg.ss_grad_H_workspace_bytes(S.disc), dtype=torch.uint8, device="cuda")
    sg.ss_grad_H(S.disc, H, lam, zero, dH, ws)
    got = dH.cpu().numpy()[0]

    ha, hb = h * r[ip] / r[ip], h * r[i] / r[i]
    q = np.arange(n_phi)
    s2 = 2 * np.sin(np.pi * q / n_phi) ** 2  # 1 - cos phi
    h2 = 0.5 * (ha * ha * np.exp(-X) + hb * hb * np.exp(X))
    x = (2 * np.sinh(X / 2) ** 2 + s2) / (4 * h2)
    assert x.min() > 256.5
    dphi = 2 * np.pi / n_phi
    c, a, coef = 1.0, 1.0, []
    for n in range(12):
        if n:
            c, a = -c * (4 * n * n - 1) / (8 * n), -a * (2 * n - 1) ** 2 / (8 * n)
        coef.append(n * c if kind == "field" else c - a)
    s = np.polyval(coef[::-1], 1 / x)
    if kind == "field":
        D = np.sqrt(2 * np.pi) / 4 * x ** -1.5 * s
        K = np.exp(-1.5 * X) / (8 * np.sqrt(np.pi)) * h2 ** -2.5 * D * (np.expm1(X) + s2)
        da, db = K.sum() * ha * np.exp(-X), K.sum() * hb * np.exp(X)
    else:
        # sample -r'^2 P: r'^2 G0(y) / (2 sqrt(pi) H); d(G0/H)/dH = E/H^2
        E = np.sqrt(np.pi / 2) * x ** -0.5 * s
        Ha, Hb = ha * r[ip], hb * r[i]
        Hm = np.sqrt(0.5 * (Ha * Ha + Hb * Hb))
        K = r[ip] ** 2 / (2 * np.sqrt(np.pi)) * E / Hm ** 2
        da, db = K.sum() * Ha * r[ip] / (2 * Hm), K.sum() * Hb * r[i] / (2 * Hm)
    want = np.zeros(n_r)
    want[ip] = -n_phi * du * dphi * da / r[ip]
    want[i] = -n_phi * du * dphi * db / r[i]
    assert np.all(got[want == 0] == 0)
    at = [ip, i]
    err = np.abs(got[at] / want[at] - 1)
    print("  ", err, flush=True)
    assert err.max() < 5e-15
