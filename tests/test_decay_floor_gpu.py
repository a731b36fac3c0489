"""A token that resets the state (a decay at or below the floor 2^-126), in the
middle of a chunk and behind 16-token blocks of strong decays: the outputs and
gradients of the tokens before and after it, against the fp64 oracle, for
decay pre-activations of any size and for a plain decay of zero."""
import numpy as np
import pytest

import paper_2509_25223_amd as rla
from oracle import preproc
from tests.gpu_util import GRAD_KEYS, TOL, dev, host, rel_err
from tests.test_parity_preproc_gpu import PRE, nudged, oracle_args, raw_inputs, to_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("z", [None, 1e4, 1e8, 1e9, 3e38], ids=str)   # None: plain gates, a decay of 0
@pytest.mark.parametrize("variant", ["rdn", "rla"])
@pytest.mark.parametrize("flags", [0, rla.RLA_FLAG_UNGATED_OUTPUT | rla.RLA_FLAG_DECAYED_RESIDUAL],
                         ids=["boxed", "variants"])
@pytest.mark.parametrize("dtype,d", [("f32", 64), ("bf16", 64), ("bf16", 128)])
def test_reset_token(device, dtype, d, flags, variant, z):
    import torch
    if z is not None:
        flags |= PRE
    lens = [64, 130]
    inp, dp = raw_inputs(406, lens, 2, d, dtype, flags, grads=True)
    for n in ("alpha_s", "alpha_r"):
        a = inp[n] = inp[n].copy()
        a[10:30] = a[10:30] + 3.0 if z is not None else 0.2   # strong decays in the blocks before
        for t in (37, 64 + 5, 64 + 100):
            a[t] = 0.0 if z is None else z
    inp = nudged(variant, inp, dp, flags, dtype)
    t = to_gpu(inp, dtype, device)
    names = ("q", "k", "v", "alpha_s", "beta", "alpha_r", "gamma")
    how = dict(cu_seqlens=t["cu"], variants=flags,
               decay_param=dev(dp, torch.float32, device) if flags & PRE else None)
    fwd, bwd = ((rla.rdn_forward, rla.rdn_backward) if variant == "rdn" else (rla.rla_forward, rla.rla_backward))
    o, S, R = fwd(*(t[n] for n in names), **how)
    g = bwd(*(t[n] for n in names), t["dO"], **how)
    torch.cuda.synchronize()
    ins, oa = [inp[n] for n in names], dict(oracle_args(inp, dp, flags), cu_seqlens=inp["cu_seqlens"])
    ref = dict(preproc.backward(variant, *ins, inp["dO"], **oa))
    ref["o"], ref["S"], ref["R"] = preproc.forward(variant, *ins, **oa)
    got = dict({key: g[key] for key in GRAD_KEYS}, o=o, S=S, R=R)
    if flags & PRE:
        ref["da"], ref["db"] = ref["ddecay_a"], ref["ddecay_b"]
        got["da"], got["db"] = g["ddecay_param"]
    errs = {}
    for key, x in got.items():
        x, want = host(x).reshape(ref[key].shape), np.array(ref[key], np.float64)
        assert np.isfinite(x).all(), key
        if key in ("dalpha_s", "dalpha_r") and z is None:   # at a decay below the floor: defined as 0
            for i in (37, 64 + 5, 64 + 100):
                assert not x[i].any()
                want[i] = 0.0
        errs[key] = rel_err(x, want)
    print("[%s %s d%d flags %d z=%s] %s" % (variant, dtype, d, flags, z,
                                            " ".join("%s=%.1e" % kv for kv in errs.items())), flush=True)
    for key, e in errs.items():
        assert e <= TOL[dtype], (key, e)
