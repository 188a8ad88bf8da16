"""Direct sums with H = h r (ring sums: the kernel between two rings taken once
per azimuth offset) at the edges of their launch shapes, against the pairwise
oracle: azimuth counts around the 8-target groups, the 64-azimuth chunks, the
staged row (1024 azimuths in float, 512 in double) and the target tile (2048
and 1024), ring counts that do not fill the last split.

Tolerances are those of the direct sums: double 1e-12 of max|g| (or |Phi|),
float 1e-5 relative RMS per fluid and component."""
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


SHAPES = [(1, 1, 1), (3, 2, 2), (40, 3, 1), (5, 7, 2), (9, 8, 1), (37, 9, 2), (6, 63, 1), (7, 64, 3), (11, 65, 2),
          (5, 200, 4), (19, 250, 2), (3, 511, 1), (3, 513, 2), (2, 1023, 1), (2, 1030, 2), (3, 2047, 1), (2, 2060, 2)]


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("what", ["field", "linear", "potential"])
@pytest.mark.parametrize("nr,nphi,nf", SHAPES)
def test_ring_sum_matches_pairwise(sg, T, nr, nphi, nf, what, dtype):
    print(f"ring sum {what} {dtype} {nr}x{nphi} nf={nf}", flush=True)
    rng = np.random.default_rng(nr * 5000 + nphi)
    td = torch.float64 if dtype == "f64" else torch.float32
    rmin, rmax = 0.5, 0.5 * np.exp(min(3.0, nr * 2 * np.pi / max(nphi, 8)))
    h = [0.05, 0.008, 0.1, 0.02][:nf]
    sig = torch.tensor(rng.uniform(0.2, 1.0, (nf, nr, nphi)), dtype=td, device="cuda")
    s64 = sig.double().cpu().numpy()
    N = nr * nphi
    cells = np.unique(np.concatenate([[0, N - 1, N // 2], rng.integers(0, N, 60)])).astype(np.int64)
    g = sg.grid(nr, nphi, rmin, rmax)
    if what == "potential":
        got = [T.potential(g, h, sig)]
        want = [O.potential_pairwise(nr, nphi, rmin, rmax, h, s64, targets=cells)]
    else:
        fl = sg.LINEAR_R if what == "linear" else 0
        got = list(T.direct(g, h, sig, flags=fl))
        want = list(O.field_pairwise(nr, nphi, rmin, rmax, h, s64, targets=cells,
                                     flags=O.LINEAR_R if fl else 0))
    got = [x.double().cpu().numpy().reshape(nf, -1)[:, cells] for x in got]
    if dtype == "f64":
        top = max(np.abs(w).max() for w in want)
        err = max(np.abs(x - w).max() for x, w in zip(got, want)) / top
        print(f"  max err / max {err:.2e}", flush=True)
        assert err < (1e-11 if N == 1 else 1e-12)
    else:
        # against the vector field: g_phi may vanish by symmetry
        for b in range(nf):
            num = sum(float(np.sum((x[b] - w[b]) ** 2)) for x, w in zip(got, want))
            den = sum(float(np.sum(w[b] ** 2)) for w in want)
            assert num <= (1e-5) ** 2 * den, (b, (num / den) ** 0.5)
