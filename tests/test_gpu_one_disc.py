"""A single disc takes its descriptor by value under a plan kept by shape: the
same call on other buffers, on two streams at once and inside a captured graph
gives what a batch of two discs (descriptors in memory) gives."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# the same sums in float32, possibly in another launch shape: a few roundings
# of the transforms (2^-24 log2(2 n_r n_phi)) against the largest |g|
TOL = 2e-6


@pytest.fixture(scope="module")
def sg():
    import paper_2506_10812_amd as sg
    return sg


def _disc(sg, T, n_r, n_phi, nf, flags, semi, rng):
    g = sg.grid(n_r, n_phi, 0.4, 2.5)
    hs = [0.05, 0.02][:nf]
    if semi:
        S = T.SemiSpectral(n_r, n_phi, 0.4, 2.5, nf, flags)
        r = 0.4 * np.exp((np.arange(n_r) + 0.5) * np.log(2.5 / 0.4) / n_r)
        S.refresh(np.array(hs)[:, None] * r[None, :] ** 1.2)
        table, f, fl = S.table, S.disc.fluids, flags | sg.SEMI_SPECTRAL
    else:
        f, fl = sg.fluids(hs), flags
        table = T.build_table(g, f, flags)
    out = []
    for _ in range(2):
        sig = torch.tensor(rng.uniform(0.1, 2.0, (nf, n_r, n_phi)), dtype=torch.float32, device="cuda")
        gr, gp = torch.full_like(sig, float("nan")), torch.full_like(sig, float("nan"))
        d = sg.make_disc(g, f, fl, sig, gr, gp, table)
        ws = torch.empty(max(1, sg.field_fft_workspace_bytes([d])), dtype=torch.uint8, device="cuda")
        out.append((d, sig, gr, gp, ws, table))
    return out


@pytest.mark.parametrize("n_r,n_phi,nf,flags,semi", [(2, 4, 1, 0, False), (4, 8, 2, 4, False), (64, 128, 1, 0, False),
                                                     (16, 2048, 2, 0, False), (512, 256, 2, 4, False),
                                                     (33, 32, 2, 0, True), (130, 64, 1, 4, True)])
def test_one_disc_equals_batch(sg, n_r, n_phi, nf, flags, semi):
    from paper_2506_10812_amd import torch_ops as T
    print(f"one disc {n_r}x{n_phi} fluids {nf} flags {flags} semi {semi}", flush=True)
    rng = np.random.default_rng(n_r * 31 + n_phi)
    sets = _disc(sg, T, n_r, n_phi, nf, flags, semi, rng)
    pair = [s[0] for s in sets]
    ws2 = torch.empty(max(1, sg.field_fft_workspace_bytes(pair)), dtype=torch.uint8, device="cuda")
    sg.field_fft(pair, ws2)
    torch.cuda.synchronize()
    ref = [(s[2].clone(), s[3].clone()) for s in sets]

    def check():
        torch.cuda.synchronize()
        for (_, _, gr, gp, _, _), (rr, rp) in zip(sets, ref):
            scale = max(float(rr.abs().max()), float(rp.abs().max()), 1e-30)
            assert float((gr - rr).abs().max()) <= TOL * scale
            assert float((gp - rp).abs().max()) <= TOL * scale
            gr.fill_(float("nan"))
            gp.fill_(float("nan"))
        torch.cuda.synchronize()

    for d, _, _, _, ws, _ in sets:
        sg.field_fft([d], ws)
    n0 = sg.field_fft_cache_entries()
    check()
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    for (d, _, _, _, ws, _), st in zip(sets, streams):
        sg.field_fft([d], ws, stream=st)
    check()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        for d, _, _, _, ws, _ in sets:
            sg.field_fft([d], ws, stream=torch.cuda.current_stream())
    for _ in range(3):
        graph.replay()
        check()
    assert sg.field_fft_cache_entries() == n0  # one plan for both sets of buffers
