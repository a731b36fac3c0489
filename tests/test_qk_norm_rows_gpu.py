"""The in-operator normalisation at row counts around its blocks (a workgroup
takes 32 rows of 128 bf16 or 64 fp32 values, 64 of 64 bf16 values, in two sets
of 4 or 8 rows a wave), with a zero row (below the norm's floor) first and last,
against the fp64 oracle."""
import numpy as np
import pytest

import paper_2509_25223_amd as rla
from oracle import preproc
from tests.gpu_util import TOL, dev, host, rel_err
from tests.test_parity_preproc_gpu import QKN, nudged, oracle_args, raw_inputs, to_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,H", [(1, 1), (3, 1), (5, 3), (16, 1), (31, 1), (11, 3), (33, 2), (65, 1)])
@pytest.mark.parametrize("dtype,d", [("f32", 64), ("bf16", 64), ("bf16", 128)])
def test_row_counts(device, dtype, d, T, H):
    import torch
    inp, dp = raw_inputs(405, [T], H, d, dtype, QKN, grads=True)
    if T > 2:
        for n in ("q", "k"):
            inp[n] = inp[n].copy()
            inp[n][0, 0] = 0.0
            inp[n][-1, -1] = 0.0
    inp = nudged("rdn", inp, dp, QKN, dtype)
    t = to_gpu(inp, dtype, device)
    args = [t[n] for n in ("q", "k", "v", "alpha_s", "beta", "alpha_r", "gamma")]
    o, _, _ = rla.rdn_forward(*args, cu_seqlens=t["cu"], variants=QKN)
    g = rla.rdn_backward(*args, t["dO"], cu_seqlens=t["cu"], variants=QKN)
    torch.cuda.synchronize()
    oa = oracle_args(inp, dp, QKN)
    ins = [inp[n] for n in ("q", "k", "v", "alpha_s", "beta", "alpha_r", "gamma")]
    ro, _, _ = preproc.forward("rdn", *ins, cu_seqlens=inp["cu_seqlens"], **oa)
    ref = preproc.backward("rdn", *ins, inp["dO"], cu_seqlens=inp["cu_seqlens"], **oa)
    assert rel_err(host(o), ro) <= TOL[dtype]
    for key in ("dq", "dk"):
        got, want = host(g[key]).reshape(ref[key].shape), ref[key].copy()
        live = np.ones(got.shape[:2], bool)
        if T > 2:   # a zero row's gradient is dx_hat 1e12 / 2: finite or infinite in bf16, not compared
            live[0, 0] = live[-1, -1] = False
        if not np.any(want[live]):
            assert not np.any(got[live])
            continue
        assert rel_err(got[live], want[live]) <= TOL[dtype], key
