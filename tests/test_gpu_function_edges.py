"""F, F' and G0 = e^x K0 on the device at the edges of their branches (power
series below 1/16, local polynomials on 8 (float: 4) intervals per octave,
asymptotic series from 256 (float: 64)): each edge and one ulp either side,
every interval's ends, the extremes of the range, infinity and NaN, against
the oracle.  Double 5e-15, float 1e-6 relative, the bars of these functions."""
import numpy as np
import pytest

import oracle as O

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def sg():
    import paper_2506_10812_amd as m
    return m


@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_function_edges(sg, dtype):
    print(f"function edges {dtype}", flush=True)
    nt = np.float64 if dtype == "f64" else np.float32
    edges = np.array([2.0 ** o * (1 + k / 8) for o in range(-5, 9) for k in range(8)] + [1e-12, 1e-4, 4e4], dtype=nt)
    x = np.unique(np.concatenate([edges, np.nextafter(edges, nt(0)), np.nextafter(edges, nt(np.inf)),
                                  np.geomspace(1e-6, 1e5, 501).astype(nt)]))
    xt = torch.tensor(x, device="cuda")
    F, dF, G = (torch.empty_like(xt) for _ in range(3))
    code = sg.F64 if dtype == "f64" else sg.F32
    sg.eval_F(xt, F, dF if dtype == "f64" else None, code)
    sg.eval_G0(xt, G, code)
    torch.cuda.synchronize()
    xd = x.astype(np.float64)
    tol = 5e-15 if dtype == "f64" else 1e-6
    for name, got, want in [("F", F, O.F(xd)), ("G0", G, O.G0(xd))] + ([("dF", dF, O.dF(xd))] if dtype == "f64" else []):
        err = np.abs(got.double().cpu().numpy() / want - 1)
        print(f"  {name}: {err.max():.2e} at x = {xd[err.argmax()]:.6g}", flush=True)
        assert err.max() < tol, name


@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_function_limits(sg, dtype):
    x = torch.tensor([float("inf"), float("nan")], dtype=torch.float64 if dtype == "f64" else torch.float32,
                     device="cuda")
    F, G = torch.empty_like(x), torch.empty_like(x)
    code = sg.F64 if dtype == "f64" else sg.F32
    sg.eval_F(x, F, None, code)
    sg.eval_G0(x, G, code)
    f, g = F.cpu().numpy(), G.cpu().numpy()
    assert f[0] == 0.0 and g[0] == 0.0 and np.isnan(f[1]) and np.isnan(g[1])
