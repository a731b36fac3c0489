"""The chunk-start states that a saving forward leaves for its backward are the
fp32 states rounded once: fp16, each 16-row x 32-column tile divided by the power
of two that brings its largest magnitude into [2^13, 2^14).  The states
themselves are the final states of forwards that end where the chunk starts (a
split at a chunk boundary gives the same bits)."""
import numpy as np
import pytest

import paper_2509_25223_amd as rla

pytestmark = pytest.mark.gpu


def saved_form(state):
    """A [d_k, d_v] state as stored: 32 columns at a time, fp16."""
    dk, dv = state.shape
    tiles = state.reshape(dk // 16, 16, dv // 32, 32)
    scale = 2.0 ** (np.floor(np.log2(np.abs(tiles).max(axis=(1, 3), keepdims=True))) - 13)
    return np.ascontiguousarray((tiles / scale).astype(np.float16).transpose(2, 0, 1, 3))


@pytest.mark.parametrize("raw", [False, True], ids=["plain", "raw"])
@pytest.mark.parametrize("d,dv", [(64, 64), (128, 128), (64, 128), (128, 64)])
@pytest.mark.parametrize("op", ["rdn", "rla"])
def test_saved_states_are_rounded_once(device, op, d, dv, raw):
    import torch
    T, H = 3 * 64 + 5, 2
    gen = torch.Generator(device).manual_seed(31)
    q, k = (torch.randn(1, T, H, d, device=device, generator=gen) for _ in range(2))
    if not raw:
        q, k = (x / x.norm(dim=-1, keepdim=True) for x in (q, k))
    v = torch.randn(1, T, H, dv, device=device, generator=gen)
    x = [t.bfloat16() for t in (q, k, v)]
    x += [torch.rand(1, T, H, device=device, generator=gen) * 0.8 + 0.1 for _ in range(4)]
    fn, code = ((rla.rdn_forward, rla.RLA_OP_RDN_BACKWARD) if op == "rdn" else
                (rla.rla_forward, rla.RLA_OP_RLA_BACKWARD))
    flags = rla.RLA_FLAG_QK_SILU_L2NORM if raw else 0
    prob = rla.make_problem(x[0], x[2], None, 1.0, None, flags)
    ws = torch.zeros(rla.rla_workspace_size(prob, code), dtype=torch.uint8, device=device)
    fn(*x, workspace=ws, save_for_backward=True, variants=flags)
    saved = ws.cpu().numpy().tobytes()
    for c in (1, 2, 3):
        _, *states = fn(*(t[:, :64 * c].contiguous() for t in x), variants=flags)
        for state in states:
            for h in range(H):
                assert saved_form(state[0, h].cpu().numpy()).tobytes() in saved, (c, h)
