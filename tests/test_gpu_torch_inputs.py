"""SGField and SGFieldSS read dense inputs in place; every other form (strided,
expanded, misaligned, lazily negated, double) gives the same bits as a clean
float32 copy of it, and no call writes to or keeps another call's tensors."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
NF, NR, NPHI = 2, 32, 64


def _forms(x):
    pad = torch.zeros(x.numel() + 1, device=x.device)
    pad[1:] = x.flatten()
    wide = torch.zeros((NF, NR, 2 * NPHI), device=x.device)
    wide[..., ::2] = x
    neg = torch.complex(torch.zeros_like(x), -x).conj().imag
    assert neg.is_neg()
    return {"dense": x.clone(), "strided": wide[..., ::2], "misaligned": pad[1:].view(x.shape), "negated": neg,
            "transposed": x.transpose(1, 2).contiguous().transpose(1, 2), "double": x.double()}


@pytest.mark.parametrize("semi", [False, True])
def test_every_form_of_input_gives_the_same_bits(semi):
    from paper_2506_10812_amd import torch_ops as T
    gen = torch.Generator(device="cpu").manual_seed(5)
    sig, lr, lp = [torch.rand((NF, NR, NPHI), generator=gen).cuda() for _ in range(3)]
    h = torch.tensor([0.05, 0.02], dtype=torch.float64, device="cuda")
    if semi:
        r = 0.4 * torch.exp((torch.arange(NR, device="cuda") + 0.5) * torch.log(torch.tensor(2.5 / 0.4)) / NR)
        h = h[:, None] * r[None, :].double()
    op = T.SGFieldSS if semi else T.SGField

    def run(s, a, b):
        s = s.detach().requires_grad_() if s.dtype == torch.float32 else s.clone().requires_grad_()
        hh = h.clone().requires_grad_()
        gr, gp = op.apply(s, hh, NR, NPHI, 0.4, 2.5)
        torch.autograd.backward([gr, gp], [a, b])
        return gr.detach(), gp.detach(), s.grad, hh.grad

    ref = run(sig, lr, lp)
    keep = [x.clone() for x in ref]
    for name, s in _forms(sig).items():
        for other, a in _forms(lr).items():
            if a.dtype != torch.float32:
                continue
            print(f"semi {semi} sigma {name} lam {other}", flush=True)
            out = run(s, a, lp)
            assert torch.equal(s.float(), sig) and torch.equal(a.contiguous(), lr)  # inputs untouched
            for x, y in zip(out, ref):
                assert torch.equal(x.float(), y.float())
    one = torch.ones((), device="cuda").expand(NF, NR, NPHI)
    for x, y in zip(run(sig, one, one), run(sig, torch.ones_like(sig), torch.ones_like(sig))):
        assert torch.equal(x, y)
    for x, y in zip(ref, keep):  # results are their callers' own
        assert torch.equal(x, y)
