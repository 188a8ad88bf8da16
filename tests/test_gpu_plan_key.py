"""Plans that sg_field_fft keeps, when the same buffers come back with other
radii: a plan may be kept only where nothing in it depends on them."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sg():
    import paper_2506_10812_amd as sg
    return sg


def _solve(sg, shared, n_r, n_phi, radii, n_discs, groups):
    """Fields of n_discs semi-spectral discs in the buffers `shared`."""
    g, f = sg.grid(n_r, n_phi, *radii), sg.fluids([0.05])
    r = radii[0] * np.exp((np.arange(n_r) + 0.5) * np.log(radii[1] / radii[0]) / n_r)
    H = torch.tensor(0.05 * r[None, :] ** 1.2, dtype=torch.float64, device="cuda")
    discs = []
    for sig, gr, gp, table in shared["discs"][:n_discs]:
        nb = sg.ss_table_bytes(g, 1, 0)
        assert 0 < nb <= table.numel()
        sg.ss_table(g, 1, H, 0, table, shared["tws"])
        gr.fill_(float("nan"))
        gp.fill_(float("nan"))
        discs.append(sg.make_disc(g, f, sg.SEMI_SPECTRAL, sig, gr, gp, table, groups))
    sg.field_fft(discs, shared["ws"])
    torch.cuda.synchronize()
    return [(gr.clone(), gp.clone()) for _, gr, gp, _ in shared["discs"][:n_discs]]


@pytest.mark.parametrize("n_discs,groups", [(2, None), (1, [0, 0])])
@pytest.mark.parametrize("first,then", [((2.0, 2.02), (2.0, 25.0)), ((2.0, 25.0), (2.0, 250.0))])
def test_semi_spectral_batches_follow_the_radii(sg, n_discs, groups, first, then):
    """The band of a mode, and with it the column that the middle pass stages,
    depends on the radii: a batch and a species disc solved in buffers that held
    a disc of other radii give what fresh buffers give.  The same kernels on the
    same numbers: equal."""
    n_r, n_phi = 96, 256
    print(f"plan key {n_discs} discs, groups {groups}, {first} then {then}", flush=True)
    ns = len(groups) if groups else 1
    rng = np.random.default_rng(5)
    sig = rng.uniform(0.1, 2.0, (2, ns, n_r, n_phi)).astype(np.float32)
    nb = max(sg.ss_table_bytes(sg.grid(n_r, n_phi, *x), 1, 0) for x in (first, then))

    def buffers():
        b = {"discs": [(torch.tensor(sig[i], device="cuda"), torch.empty((1, n_r, n_phi), device="cuda"),
                        torch.empty((1, n_r, n_phi), device="cuda"),
                        torch.empty(nb, dtype=torch.uint8, device="cuda")) for i in range(2)]}
        g = sg.grid(n_r, n_phi, *first)
        b["tws"] = torch.empty(sg.ss_table_workspace_bytes(g, 1), dtype=torch.uint8, device="cuda")
        b["ws"] = torch.zeros(1 << 22, dtype=torch.uint8, device="cuda")
        return b

    shared = buffers()
    _solve(sg, shared, n_r, n_phi, first, n_discs, groups)
    got = _solve(sg, shared, n_r, n_phi, then, n_discs, groups)
    want = _solve(sg, buffers(), n_r, n_phi, then, n_discs, groups)
    for (a, b), (x, y) in zip(got, want):
        assert bool(torch.isfinite(x).all()) and float(x.abs().max()) > 0
        assert torch.equal(a, x) and torch.equal(b, y)


@pytest.mark.parametrize("n_discs", [1, 2])
def test_fft_plans_serve_any_radii(sg, n_discs):
    """Nothing in an FFT-path plan depends on the radii: a grid that moves
    between calls (a table per step, the same buffers) takes no further plan."""
    from paper_2506_10812_amd import torch_ops as T
    print(f"plan key fft {n_discs}", flush=True)
    f, sig = sg.fluids([0.05]), torch.rand((n_discs, 1, 16, 32), device="cuda")
    out, want = torch.empty((2, n_discs, 1, 16, 32), device="cuda"), []
    ws = torch.empty(1 << 20, dtype=torch.uint8, device="cuda")
    table = T.build_table(sg.grid(16, 32, 0.4, 2.5), f)
    n = []
    for r_max in (2.5, 2.6, 2.7, 25.0):
        g = sg.grid(16, 32, 0.4, r_max)
        table.copy_(T.build_table(g, f))
        sg.field_fft([sg.make_disc(g, f, 0, sig[i], out[0, i], out[1, i], table) for i in range(n_discs)], ws)
        torch.cuda.synchronize()
        n.append(sg.field_fft_cache_entries())
        want.append(out.clone())
        assert bool(torch.isfinite(out).all())
    assert n == [n[0]] * len(n)
    assert all(not torch.equal(want[0], w) for w in want[1:])  # the tables were used
