"""H = h r sums on either side of the rule that takes rings of few cells cell
by cell (1000 rings, 700 for four fluids with one azimuth, 1500 for the
potential; 8, 6 or 5 azimuths), against the oracle's pair sums at every 97th
cell.  Double 1e-12 of max|g| (or |Phi|), float 1e-5 relative RMS over both
components: the bars of the ring sums."""
import numpy as np
import pytest

import oracle as O

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind,dtype,nr,nphi,nf", [
    ("field", "f32", 999, 1, 2), ("field", "f64", 699, 1, 4), ("field", "f64", 700, 1, 4), ("field", "f32", 1000, 1, 2), ("field", "f32", 1000, 7, 1), ("field", "f32", 1000, 8, 1),
    ("field", "f64", 1000, 1, 1), ("field", "f64", 1000, 5, 1), ("field", "f64", 1000, 6, 1),
    ("field LINEAR_R", "f64", 1003, 3, 1), ("field INDIRECT", "f32", 1000, 4, 3),
    ("potential", "f32", 1500, 4, 2), ("potential", "f64", 1499, 4, 1), ("potential", "f64", 1500, 5, 1),
    ("potential", "f64", 1500, 1, 4)])
def test_few_azimuths(kind, dtype, nr, nphi, nf):
    import paper_2506_10812_amd as sg
    from paper_2506_10812_amd import torch_ops as T
    print(f"few azimuths {kind} {dtype} {nr}x{nphi} nf={nf}", flush=True)
    h = [0.05, 0.02, 0.08, 0.03][:nf]
    rng = np.random.default_rng(nr + nphi)
    sig = rng.uniform(0.5, 1.5, (nf, nr, nphi)).astype(np.float32 if dtype == "f32" else np.float64)
    flags = sum(getattr(sg, k) for k in kind.split() if k.isupper())
    g = sg.grid(nr, nphi, 0.2, 5.0)
    st = torch.tensor(sig, device="cuda")
    at = np.arange(0, nr * nphi, 97, dtype=np.int32)
    s64 = sig.astype(np.float64)
    if kind == "potential":
        got = [T.potential(g, h, st, None, flags)]
        want = [O.potential_pairwise(nr, nphi, 0.2, 5.0, h, s64, targets=at)]
    else:
        got = T.direct(g, h, st, None, flags)
        want = list(O.field_pairwise(nr, nphi, 0.2, 5.0, h, s64, targets=at,
                                     flags=O.LINEAR_R if "LINEAR_R" in kind else 0))
        if "INDIRECT" in kind:
            AB = O.indirect(nr, nphi, 0.2, 5.0, h, s64)
            ir, ip = O.indirect_field(nr, nphi, AB)
            want = [w + np.asarray(x).reshape(-1)[at] for w, x in zip(want, (ir, ip))]
    torch.cuda.synchronize()
    got = np.stack([a.double().cpu().numpy().reshape(nf, -1)[:, at] for a in got])
    want = np.stack([np.asarray(w).reshape(nf, -1) for w in want])
    if dtype == "f64":
        err, bar = np.abs(got - want).max() / np.abs(want).max(), 1e-12
    else:
        err, bar = np.sqrt(((got - want) ** 2).sum() / (want ** 2).sum()), 1e-5
    print(f"  {err:.2e}", flush=True)
    assert err < bar
