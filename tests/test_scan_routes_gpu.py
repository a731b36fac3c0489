"""The scans' routes by head dimensions, output type and row type: plain and
normalised (SiLU + L2) rows, every supported (d_k, d_v), fp32 and bf16
outputs, ragged packed sequences, through a saving forward and its backward,
against the fp64 oracle.  bf16 outputs are compared with one output rounding
(2^-8 of the value) set aside."""
import numpy as np
import pytest

import datagen
import oracle
import paper_2509_25223_amd as rla
from oracle import preproc
from tests.gpu_util import GRAD_KEYS, TOL, dev, host, rel_err

pytestmark = pytest.mark.gpu

LENS = [1, 64, 0, 130, 63, 257]


def err(x, ref, rounded):
    if not rounded:
        return rel_err(x, ref)
    rms = float(np.sqrt(np.mean(ref * ref)))
    return float(np.max(np.maximum(np.abs(x - ref) - 2.0 ** -8 * np.abs(ref), 0.0))) / rms


@pytest.mark.parametrize("variant", ["rdn", "rla"])
@pytest.mark.parametrize("raw", [False, True], ids=["plain", "raw"])
@pytest.mark.parametrize("dk,dv", [(64, 64), (64, 128), (128, 64), (128, 128)])
@pytest.mark.parametrize("out", ["f32", "bf16"])
def test_forward_and_backward(device, variant, raw, dk, dv, out):
    import torch
    H = 3
    wl = datagen.small(variant + "_fwdbwd", "bf16", LENS, H=H, d=dk, dv=dv)
    inp = datagen.make_inputs(wl, seed=601)
    if raw:
        rng = np.random.default_rng(602)
        for n in ("q", "k"):
            inp[n] = datagen.round_to_bf16(rng.standard_normal(inp[n].shape).astype(np.float32))
    S0, R0 = datagen.random_states(61, len(LENS), H, dk, dv)
    dSf, dRf = datagen.random_states(62, len(LENS), H, dk, dv, scale=1.0)
    qk = (inp["q"], inp["k"]) if not raw else tuple(preproc.qk_transform(inp[n]) for n in ("q", "k"))
    gates = [inp[n] for n in ("alpha_s", "beta", "alpha_r", "gamma")]
    cu = inp["cu_seqlens"]
    v, _ = oracle.nudge_margin(variant, *qk, inp["v"], *gates, clip=1.0, S0=S0, R0=R0, cu_seqlens=cu,
                               margin=2e-2, grid="bf16", flags=0)
    inp["v"] = v.astype(np.float32)
    ref = oracle.backward(variant, *qk, inp["v"], *gates, inp["dO"], S0=S0, R0=R0, dS_final=dSf, dR_final=dRf,
                          cu_seqlens=cu)
    ref = dict(ref)
    ref["o"], ref["S"], ref["R"] = oracle.forward(variant, *qk, inp["v"], *gates, S0=S0, R0=R0, cu_seqlens=cu)
    if raw:
        ref.update({"d" + n: preproc.qk_transform_grad(inp[n], ref["d" + n]) for n in ("q", "k")})

    q, k, vd, dO = (dev(inp[n], torch.bfloat16, device) for n in ("q", "k", "v", "dO"))
    g = [dev(x, torch.float32, device) for x in gates]
    f = lambda x: dev(x, torch.float32, device)   # noqa: E731
    how = dict(cu_seqlens=torch.from_numpy(cu.astype(np.int32)).to(device), S0=f(S0), R0=f(R0),
               out_dtype=torch.float32 if out == "f32" else torch.bfloat16,
               variants=rla.RLA_FLAG_QK_SILU_L2NORM if raw else 0)
    fwd, bwd, op = ((rla.rdn_forward, rla.rdn_backward, rla.RLA_OP_RDN_BACKWARD) if variant == "rdn" else
                    (rla.rla_forward, rla.rla_backward, rla.RLA_OP_RLA_BACKWARD))
    prob = rla.make_problem(q, vd, how["cu_seqlens"], 1.0, how["out_dtype"], how["variants"])
    ws = torch.empty(rla.rla_workspace_size(prob, op), dtype=torch.uint8, device=device)
    o1, S1, R1 = fwd(q, k, vd, *g, **how)
    o, S, R = fwd(q, k, vd, *g, workspace=ws, save_for_backward=True, **how)
    grads = bwd(q, k, vd, *g, dO, dS_final=f(dSf), dR_final=f(dRf), workspace=ws, use_saved=True, **how)
    torch.cuda.synchronize()
    assert torch.equal(o, o1) and torch.equal(S, S1) and torch.equal(R, R1)   # saving or not: the same bits
    got = dict({key: grads[key] for key in GRAD_KEYS}, o=o, S=S, R=R)
    errs = {key: err(host(t).reshape(ref[key].shape), np.asarray(ref[key], np.float64),
                     out == "bf16" and key in ("o", "dq", "dk", "dv")) for key, t in got.items()}
    print("[%s %s dk%d dv%d %s] %s" % (variant, "raw" if raw else "plain", dk, dv, out,
                                       " ".join("%s=%.1e" % kv for kv in errs.items())), flush=True)
    for key, e in errs.items():
        assert e <= TOL["bf16"], (key, e)
