"""Direct sums on a uniform radial grid whose rings are close against their
radius: the rings' distances are (i - k) dr, not differences of rounded radii.
Float against the double sum of the same call, 1e-5 relative RMS per fluid and
component (the bar of the float sums); double against the oracle, 1e-12 of
max|g|."""
import numpy as np
import pytest

import oracle as O

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cells", [False, True])
@pytest.mark.parametrize("nr,nphi,nf,ratio", [(30, 40, 2, 1.01), (20, 33, 1, 1.0005), (1001, 3, 1, 1.2)])
def test_thin_annulus(nr, nphi, nf, ratio, cells):
    import paper_2506_10812_amd as sg
    from paper_2506_10812_amd import torch_ops as T
    print(f"thin annulus {nr}x{nphi} nf={nf} ratio {ratio} cells {cells}", flush=True)
    lo, hi, h = 20.0, 20.0 * ratio, [0.05, 0.02][:nf]
    rng = np.random.default_rng(nr)
    sig = rng.uniform(0.5, 1.5, (nf, nr, nphi)).astype(np.float32)
    H = None
    if cells:
        r = lo + (np.arange(nr) + 0.5) * (hi - lo) / nr
        H = (np.array(h)[:, None, None] * r[None, :, None] * rng.uniform(0.9, 1.1, (nf, nr, nphi))).astype(np.float32)
    g = sg.grid(nr, nphi, lo, hi)

    def call(dt):
        return [x.double().cpu().numpy().reshape(nf, -1)
                for x in T.direct(g, h, torch.tensor(sig, device="cuda").to(dt),
                                  None if H is None else torch.tensor(H, device="cuda").to(dt), sg.LINEAR_R)]

    single, double = call(torch.float32), call(torch.float64)
    at = np.arange(0, nr * nphi, 29, dtype=np.int32)
    want = O.field_pairwise(nr, nphi, lo, hi, h, sig.astype(np.float64), H=None if H is None else H.astype(np.float64),
                            targets=at, flags=O.LINEAR_R)
    top = max(np.abs(w).max() for w in want)
    for a, b, w in zip(single, double, want):
        e64 = np.abs(b[:, at] - np.asarray(w)).max() / top
        e32 = [float(np.sqrt(((a[f] - b[f]) ** 2).sum() / (b[f] ** 2).sum())) for f in range(nf)]
        print(f"  double {e64:.1e}, float {e32}", flush=True)
        assert e64 < 1e-12 and max(e32) < 1e-5
