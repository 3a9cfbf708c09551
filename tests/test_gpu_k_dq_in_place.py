"""dQ written over an input of the backward: the buffer of Q, dO or (bfloat16 or
float32) O holds the input when the call starts and dQ when it ends, whatever
passes the list takes, and dQ, dK and dV are those of a call with buffers of its
own.  dK/dV take P and dS from the same lse and Delta up to the order of Delta's
float32 sum of D products: |dDelta| <= D * 2^-24 * sum |dO O|, far below the
bfloat16 rounding of dS (2^-9), so the two calls agree within one rounding of dS
and one of the result on each side, 2^-8 in the 2-norm."""
import functools

import numpy as np
import pytest

from paper_2609_22755_amd import nsp
from paper_2609_22755_amd.workloads import draw_attention_inputs, small_worklist

from gpu_util import rel_l2, report, require_gpu, run_attention, to_np

pytestmark = pytest.mark.gpu

LISTS = {
    # name: (lengths, hq, hkv, head_dim): both passes in one launch; two key
    # groups and split key tiles; 128-row units, one workgroup a unit and
    # persistent; persistent 256-row units
    "small": ([130, 1, 64], 4, 2, 128),
    "keys": ([1280, 130], 4, 2, 64),
    "short": ([300] * 20 + [33], 8, 2, 128),
    "short_persistent": ([700] * 130, 8, 2, 64),
    "long": ([2560] * 14, 8, 2, 128),
}


@functools.lru_cache(maxsize=1)
def inputs(name):
    lengths, hq, hkv, D = LISTS[name]
    wl = small_worklist(lengths, hq, hkv, D)
    return wl, draw_attention_inputs(wl, 700 + len(name))


@pytest.mark.parametrize("over", ["q", "dout", "o", "o32"])
@pytest.mark.parametrize("name", sorted(LISTS))
def test_dq_over_an_input(name, over):
    import torch
    require_gpu()
    wl, inp = inputs(name)
    scale = 1.0 / np.sqrt(wl.head_dim)
    dt = torch.float32 if over == "o32" else torch.bfloat16
    ref = run_attention(wl, *inp, scale, o_dtype=dt, g_dtype=dt)
    q, k, v, do = (nsp.to_device_bf16(x) for x in inp)
    o = ref["o"].clone()
    dq = {"q": q, "dout": do, "o": o, "o32": o}[over]
    dk, dv = torch.full_like(ref["dk"], float("nan")), torch.full_like(ref["dv"], float("nan"))
    nsp.nsp_varlen_attn_bwd(wl, q, k, v, o, do, ref["lse"], dq, dk, dv, ref["ws"], scale)
    torch.cuda.synchronize()
    errs = {n: rel_l2(to_np(t), to_np(ref[n])) for n, t in (("dq", dq), ("dk", dk), ("dv", dv))}
    report(f"dq over {over}, {name}", **errs)
    assert max(errs.values()) <= 2.0 ** -8
    if name == "small":
        assert all(torch.equal(t, ref[n]) for n, t in (("dq", dq), ("dk", dk), ("dv", dv)))
