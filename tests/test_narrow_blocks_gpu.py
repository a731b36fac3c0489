"""A forward call that does not save takes 16 value columns per workgroup when
its grid is small (sequences x heads x d_v / 16 <= 256) and 32 otherwise: the
same sequence alone and in a batch past that line gives the same bits."""
import pytest

import paper_2509_25223_amd as rla

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T", [1, 63, 65, 128, 200])
@pytest.mark.parametrize("d,dv", [(128, 128), (64, 64), (64, 128), (128, 64)])
@pytest.mark.parametrize("op", ["rdn", "rla"])
@pytest.mark.parametrize("raw,out", [(False, "f32"), (False, "bf16"), (True, "f32"), (True, "bf16")])
def test_alone_as_in_a_batch(device, op, raw, out, d, dv, T):
    import torch
    H = 2
    n = 256 * 16 // (H * dv) + 1   # one sequence past the line
    gen = torch.Generator(device).manual_seed(T + d + dv)
    q, k = (torch.randn(n, T, H, d, device=device, generator=gen) for _ in range(2))
    if not raw:
        q, k = (x / x.norm(dim=-1, keepdim=True) for x in (q, k))
    v = torch.randn(n, T, H, dv, device=device, generator=gen)
    q, k, v = (x.bfloat16() for x in (q, k, v))
    gates = [torch.rand(n, T, H, device=device, generator=gen) * 0.8 + 0.1 for _ in range(4)]
    S0, R0 = (0.1 * torch.randn(n, H, d, dv, device=device, generator=gen) for _ in range(2))
    fn = rla.rdn_forward if op == "rdn" else rla.rla_forward
    how = dict(variants=rla.RLA_FLAG_QK_SILU_L2NORM if raw else 0,
               out_dtype=torch.float32 if out == "f32" else torch.bfloat16)
    many = fn(q, k, v, *gates, S0=S0, R0=R0, **how)
    one = fn(q[:1], k[:1], v[:1], *(g[:1] for g in gates), S0=S0[:1], R0=R0[:1], **how)
    torch.cuda.synchronize()
    for a, b in zip(one, many):
        assert torch.equal(a, b[:1])
