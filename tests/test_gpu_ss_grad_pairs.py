"""dL/dH(r) by ring pairs (both rows and both derivatives of a pair from one
transform) against central differences of the loss through tables rebuilt at
H +- eps in one direction, over odd ring counts, the smallest grids, several
fluids, the indirect term, the excluded own cell, a uniform grid and the
potential.  The table holds floats: eps 1e-3 of H puts the difference's own
error at 2^-24 / 1e-3 of sum |lam g| (1e-4 of it) and its truncation at 1e-6."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
TOL = 1e-4


@pytest.mark.parametrize("nr,nphi,nf,flag", [(1, 4, 1, ""), (2, 8, 2, ""), (17, 4, 1, ""), (15, 16, 3, "INDIRECT"),
                                             (33, 64, 4, ""), (33, 256, 1, "SELF_CELL_EXCLUDE"),
                                             (47, 512, 2, "LINEAR_R"), (16, 32, 2, "LINEAR_R"),
                                             (40, 256, 2, "POTENTIAL"), (129, 1024, 1, "INDIRECT"),
                                             (9, 2048, 1, ""), (70, 512, 1, "SS_FULL")])
def test_pairs_against_central_differences(nr, nphi, nf, flag):
    import paper_2506_10812_amd as sg
    from paper_2506_10812_amd import torch_ops as T
    print(f"dL/dH pairs {nr}x{nphi} nf={nf} {flag}", flush=True)
    flags = getattr(sg, flag) if flag else 0
    S = T.SemiSpectral(nr, nphi, 0.4, 2.5, nf, flags)
    gen = torch.Generator(device="cpu").manual_seed(nr * 7 + nphi)
    x = (torch.arange(nr, dtype=torch.float64) + 0.5) / nr
    r = 0.4 + 2.1 * x if flag == "LINEAR_R" else 0.4 * (2.5 / 0.4) ** x
    H = torch.stack([h * r ** 1.2 for h in (0.05, 0.08, 0.03, 0.06)[:nf]]).cuda()
    S.sigma.copy_(torch.rand((nf, nr, nphi), generator=gen))
    lr, lp = [torch.rand((nf, nr, nphi), generator=gen).cuda() for _ in range(2)]
    v = torch.rand((nf, nr), generator=gen, dtype=torch.float64).cuda() * H

    def loss(h):
        S.refresh(h)
        S.run()
        torch.cuda.synchronize()
        a, b = lr.double() * S.g_r.double(), lp.double() * S.g_phi.double()
        if flag == "POTENTIAL":
            b = torch.zeros_like(b)
        return float(a.sum() + b.sum()), float(a.abs().sum() + b.abs().sum())

    eps = 1e-3
    (up, mag), (down, _) = loss(H + eps * v), loss(H - eps * v)
    S.refresh(H)
    dH = torch.full((nf, nr), float("nan"), dtype=torch.float64, device="cuda")
    ws = torch.full((sg.ss_grad_H_workspace_bytes(S.disc),), 255, dtype=torch.uint8, device="cuda")
    sg.ss_grad_H(S.disc, H, lr, lp, dH, ws)
    torch.cuda.synchronize()
    got, want = float((dH * v).sum()), (up - down) / (2 * eps)
    print(f"  {got:.8e} {want:.8e} of {mag:.3e}", flush=True)
    assert abs(got - want) <= TOL * mag
