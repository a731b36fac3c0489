"""A decoding call stages its tokens in groups of 8: calls of T tokens around
the group size give the bits of T single-token calls."""
import pytest

import paper_2509_25223_amd as rla

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T", [2, 5, 7, 8, 9, 17])
@pytest.mark.parametrize("dtype,d,dv", [("bf16", 128, 128), ("bf16", 64, 128), ("f32", 64, 64)])
@pytest.mark.parametrize("op", ["rdn", "rla"])
@pytest.mark.parametrize("flags", [0, rla.RLA_FLAG_QK_SILU_L2NORM | rla.RLA_FLAG_GATE_PREACT], ids=["plain", "raw"])
def test_tokens_at_once(device, op, dtype, d, dv, T, flags):
    import torch
    B, H = 3, 2
    td = torch.bfloat16 if dtype == "bf16" else torch.float32
    gen = torch.Generator(device).manual_seed(T)
    q, k = (torch.randn(B, T, H, d, device=device, generator=gen) for _ in range(2))
    if not flags:
        q, k = (x / x.norm(dim=-1, keepdim=True) for x in (q, k))
    x = [t.to(td) for t in (q, k, torch.randn(B, T, H, dv, device=device, generator=gen))]
    x += [torch.rand(B, T, H, device=device, generator=gen) * 0.8 + 0.1 for _ in range(4)]
    S, R = (0.1 * torch.randn(B, H, d, dv, device=device, generator=gen) for _ in range(2))
    how = dict(out_dtype=td, variants=flags,
               decay_param=torch.rand(2, H, device=device, generator=gen) + 0.1 if flags else None)
    fn = rla.rdn_decode if op == "rdn" else rla.rla_decode
    o, So, Ro = fn(*x, S_in=S, R_in=R, **how)
    one = []
    for t in range(T):
        ot, S, R = fn(*(y[:, t:t + 1].contiguous() for y in x), S_in=S, R_in=R, **how)
        one.append(ot)
    torch.cuda.synchronize()
    assert torch.equal(o, torch.cat(one, 1))
    assert torch.equal(So, S) and torch.equal(Ro, R)
