"""sg_kernel_table spectra on grids whose rows fall into several sample counts
(rows |X| apart from the origin take M azimuths, M |X| >= 80), with derivative
spectra, one to four groups (several launches of items) and the own cell
dropped, against the numpy FP64 FFT of the oracle's samples at every azimuth:
1e-6 of the largest value (float rounding), the bar of the table."""
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


def al(x):
    return (x + 255) // 256 * 256


CASES = [(64, 512, 2, 25.0, "WITH_DH"), (16, 2048, 1, 8.0, ""), (128, 256, 2, 60.0, ""), (32, 1024, 1, 1.4, "WITH_DH"),
         (2, 4, 4, 3.0, "WITH_DH"), (8, 128, 4, 12.0, "WITH_DH"), (256, 64, 1, 25.0, "SELF_CELL_EXCLUDE"),
         (2048, 8, 1, 30.0, "")]


@pytest.mark.parametrize("nr,nphi,nf,ratio,kind", CASES)
def test_table_rows_match_numpy(sg, T, nr, nphi, nf, ratio, kind):
    print(f"table rows {nr}x{nphi} nf={nf} ratio={ratio} {kind}", flush=True)
    rmin, rmax = 0.3, 0.3 * ratio
    h = [0.05, 0.008, 0.1, 0.02][:nf]
    flags = getattr(sg, kind) if kind else 0
    tab = T.build_table(sg.grid(nr, nphi, rmin, rmax), sg.fluids(h), flags)
    raw = tab.cpu().numpy()
    _, _, du, dphi = O.grid(nr, nphi, rmin, rmax)
    npair, ncol, kk = nf * nf, nphi // 2 + 1, nr + 1
    o = al(al(al(496) + 8 * 2 * nr) + 8 * nphi)
    spec = raw[o:o + 8 * (ncol + 1) * npair * 2 * kk].view(np.complex64).reshape(ncol + 1, npair, 2, kk)
    o = al(o + 8 * (ncol + 1) * npair * 2 * kk)
    dspec = None
    if kind == "WITH_DH":
        dspec = raw[o:o + 8 * ncol * npair * 4 * kk].view(np.complex64).reshape(ncol, npair, 2, 2, kk)
    p = np.arange(2 * nr)
    X = np.where(p < nr, p, p - 2 * nr) * du
    XX, QQ = np.meshgrid(X, np.arange(nphi) * dphi, indexing="ij")
    scale = -du * dphi / (2 * nr * nphi)
    for a in range(nf):
        for b in range(nf):
            for which in range(3 if dspec is not None else 1):
                K = [k.reshape(2 * nr, nphi) for k in O.conv_kernels(XX.ravel(), QQ.ravel(), h[a], h[b], which)]
                for k in K:
                    k[nr] = 0
                    k[0, 0] = 0
                if kind != "SELF_CELL_EXCLUDE":
                    K[0][0, 0] = O.self_cell(h[a], h[b], du, dphi, which)
                for c in range(2):
                    ref = np.fft.fft2(K[c])[:nr + 1, :ncol].T * scale
                    got = spec[:ncol, a * nf + b, c] if which == 0 else dspec[:, a * nf + b, which - 1, c]
                    err = np.abs(got - ref).max() / np.abs(ref).max()
                    assert err < 1e-6, (a, b, which, c, err)
    k0, kn = spec[0, :, 0], spec[ncol - 1, :, 0]
    assert np.array_equal(spec[ncol, :, 0], ((k0 + kn) * np.float32(0.5)).astype(np.complex64))
    assert np.array_equal(spec[ncol, :, 1], ((k0 - kn) * np.float32(0.5)).astype(np.complex64))
