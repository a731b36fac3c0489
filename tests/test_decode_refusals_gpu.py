"""Decoding refuses what does not fit its operands, naming it, and takes calls
that leave optional operands out."""
import pytest

import paper_2509_25223_amd as rla

pytestmark = pytest.mark.gpu


def operands(device):
    import torch
    B, T, H, d = 2, 1, 3, 64
    x = dict(zip("qkv", (torch.randn(B, T, H, d, device=device).bfloat16() for _ in range(3))))
    x.update({n: torch.rand(B, T, H, device=device) for n in ("alpha_s", "beta", "alpha_r", "gamma")})
    x.update({n: torch.randn(B, H, d, d, device=device) for n in ("S_in", "R_in", "S_out", "R_out")})
    x["out"] = torch.empty(B, T, H, d, device=device)
    return x


BAD = {
    "shape k": ("k", lambda t: t[..., :32].contiguous(), ValueError),
    "shape v": ("v", lambda t: t[:1].contiguous(), ValueError),
    "shape gate": ("beta", lambda t: t[..., None].contiguous(), ValueError),
    "shape state": ("R_in", lambda t: t[:1].contiguous(), ValueError),
    "shape out": ("out", lambda t: t[:1].contiguous(), ValueError),
    "dtype k": ("k", lambda t: t.float(), TypeError),
    "dtype gate": ("gamma", lambda t: t.double(), TypeError),
    "dtype state": ("S_out", lambda t: t.half(), TypeError),
    "dtype out": ("out", lambda t: t.bfloat16(), TypeError),
    "stride": ("S_in", lambda t: t.transpose(-1, -2), ValueError),
    "device": ("v", lambda t: t.cpu(), ValueError),
    "missing": ("alpha_r", lambda t: None, ValueError),
}


@pytest.mark.parametrize("case", list(BAD))
def test_refused(device, case):
    name, change, error = BAD[case]
    x = operands(device)
    x[name] = change(x[name])
    with pytest.raises(error, match=name):
        rla.rdn_decode(**x)


def test_optional_operands(device):
    import torch
    x = operands(device)
    x["S_in"].zero_()
    x["R_in"].zero_()
    want = [t.clone() for t in rla.rdn_decode(**x)]
    got = rla.rdn_decode(*(x[n] for n in ("q", "k", "v", "alpha_s", "beta", "alpha_r", "gamma")))
    torch.cuda.synchronize()
    for a, b in zip(got, want):
        assert torch.equal(a, b)
