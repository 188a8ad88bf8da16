"""F and G0 = e^x K0 on the device over the whole range of normal numbers of
each type, against their leading terms where these are exact to the type:
below 1e-12 (float 1e-8), with K0 = -(ln(x/2) + gamma), F = 1/x + 1 - K0 and
G0 = (1 + x) K0, both to x^2 ln x; above 1e16 (float 1e8) F = sqrt(2 pi)/4
x^{-3/2} and G0 = sqrt(pi/(2x)), both to 1/x.  The bars are those of the
functions (double 5e-15, float 1e-6)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_function_range(dtype):
    import paper_2506_10812_amd as sg
    print(f"function range {dtype}", flush=True)
    nt, small, tol = (np.float64, 1e-12, 5e-15) if dtype == "f64" else (np.float32, 1e-8, 1e-6)
    info = np.finfo(nt)
    x = np.concatenate([np.geomspace(4 * float(info.tiny), small, 400), np.geomspace(1e16 if dtype == "f64" else 1e8,
                                                                                   0.9 * float(info.max), 400)]).astype(nt)
    xt = torch.tensor(x, device="cuda")
    F, G = torch.empty_like(xt), torch.empty_like(xt)
    code = sg.F64 if dtype == "f64" else sg.F32
    sg.eval_F(xt, F, None, code)
    sg.eval_G0(xt, G, code)
    torch.cuda.synchronize()
    xl = x.astype(np.longdouble)
    lo = x < 1
    K0 = -(np.log(xl / 2) + np.longdouble("0.57721566490153286061"))
    wF = np.where(lo, 1 / xl + 1 - K0, np.sqrt(2 * np.pi) / 4 / (xl * np.sqrt(xl)))
    wG = np.where(lo, (1 + xl) * K0, np.sqrt(np.longdouble(np.pi) / 2 / xl))
    for name, got, want in (("F", F, wF), ("G0", G, wG)):
        g = got.cpu().numpy().astype(np.longdouble)
        err = np.abs(g - want)
        bad = ~(err <= np.maximum(tol * np.abs(want), 2 * float(info.tiny)))  # results below the normal numbers: absolute
        assert not bad.any(), (name, x[bad][[0, -1]], g[bad][[0, -1]], want[bad][[0, -1]])
