"""The kinds of forward / dQ units: 256 query rows by eight waves, 128 rows by
four (short units), 128 rows in two key groups (lists that leave compute units
idle), at the sizes where one can go wrong: edges of 32, 128 and 256 rows and
of 32 and 64 keys, rows whose second key group is empty, both head widths and
output types, against the float64 oracle; and the same items beside long ones,
in a list that takes 256-row units: 128-row units give the same bits, two key
groups the same P (both groups scale it by the maxima of the first 32 keys, which
no later score of these inputs passes by 2^8) in sums of another order.  A row's
sum of n <= 1280 float32 terms of random sign is off by about sqrt(n) * 2^-24 of
sum |P V|, which is about sqrt(n) times |O|: n * 2^-24 < 8e-5 in all, and a
bf16 P of another scale would be 1e-3."""
import dataclasses

import numpy as np
import pytest

from paper_2609_22755_amd import nsp
from paper_2609_22755_amd.workloads import draw_attention_inputs, small_worklist

from gpu_util import (FWD_MAX_ABS, FWD_REL_L2, GRAD_REL_L2, LSE_MAX_ABS, max_abs, oracle_full, rel_l2, report,
                      require_gpu, run_attention, to_np)

pytestmark = pytest.mark.gpu

CASES = {
    # name: (lengths, sp, hq, hkv, head_dim, the list takes two key groups)
    "short_edges": ([1, 31, 32, 33, 63, 64, 65, 96, 127, 128, 129, 160, 255, 256, 257, 300], None, 8, 2, 128, False),
    "short_edges_d64": ([1, 32, 33, 64, 65, 128, 129, 255, 256, 257], None, 8, 2, 64, False),
    "keys_one": ([1153], None, 4, 1, 128, True),
    "keys_edges": ([1024, 1057, 33, 1], None, 4, 2, 128, True),
    "keys_d64": ([1280, 130, 64], None, 4, 2, 64, True),
}


def padded(wl, lengths):
    """The list with more items behind its own."""
    k = len(lengths)
    return dataclasses.replace(
        wl, lengths=np.concatenate([wl.lengths, np.array(lengths, np.int32)]),
        sp=np.concatenate([wl.sp, np.ones(k, np.int32)]),
        q_heads=np.concatenate([wl.q_heads, np.tile([[0, wl.hq_total]], (k, 1))]),
        kv_heads=np.concatenate([wl.kv_heads, np.tile([[0, wl.hkv_total]], (k, 1))]))


@pytest.mark.parametrize("name", sorted(CASES))
def test_unit_kinds(name):
    import torch
    require_gpu()
    lengths, sp, hq, hkv, D, keys = CASES[name]
    wl = small_worklist(lengths, hq, hkv, D, sp=sp)
    inp = draw_attention_inputs(wl, 500 + len(name))
    scale = 1.0 / np.sqrt(D)
    ref = oracle_full(wl, *inp, scale)
    f32 = run_attention(wl, *inp, scale, o_dtype=torch.float32, g_dtype=torch.float32)
    b16 = run_attention(wl, *inp, scale)
    errs = dict(o=rel_l2(to_np(f32["o"]), ref["o"]), o_max=max_abs(to_np(f32["o"]), ref["o"]),
                lse=max_abs(to_np(f32["lse"]), ref["lse"]), dq=rel_l2(to_np(b16["dq"]), ref["dq"]),
                dq32=rel_l2(to_np(f32["dq"]), ref["dq"]))
    report(f"kinds {name}", **errs)
    assert errs["o"] <= FWD_REL_L2 and errs["o_max"] <= FWD_MAX_ABS and errs["lse"] <= LSE_MAX_ABS
    assert errs["dq"] <= GRAD_REL_L2 and errs["dq32"] <= GRAD_REL_L2
    assert torch.equal(b16["o"].view(torch.int16), f32["o"].to(torch.bfloat16).view(torch.int16))
    big = padded(wl, [8192] * 4)
    q, k, v, do = (nsp.to_device_bf16(x) for x in inp)

    def wide(t, n):
        return torch.cat([t, torch.zeros(n - t.numel(), dtype=t.dtype, device="cuda")])

    x = [wide(q, big.q_elems()), wide(k, big.kv_elems()), wide(v, big.kv_elems())]
    o = torch.full((big.q_elems(),), float("nan"), dtype=torch.float32, device="cuda")
    lse = torch.full((big.lse_elems(),), float("nan"), dtype=torch.float32, device="cuda")
    nsp.nsp_varlen_attn_fwd(big, *x, o, lse, scale)
    torch.cuda.synchronize()
    o, lse = o[:q.numel()], lse[:f32["lse"].numel()]
    if keys:
        err = rel_l2(to_np(o), to_np(f32["o"]))
        report(f"kinds {name}: two key groups against one", o=err)
        assert not torch.equal(o, f32["o"]), "the list does not take two key groups"
        assert err <= 1280 * 2.0 ** -24 and max_abs(to_np(lse), to_np(f32["lse"])) <= 1e-5
    else:
        assert torch.equal(o.view(torch.int32), f32["o"].view(torch.int32))
        assert torch.equal(lse.view(torch.int32), f32["lse"].view(torch.int32))


PERSISTENT = {
    # more units than the compute units hold workgroups, in all three passes of
    # the first three lists (checked on the host, in native/split_checks.cpp); two
    # key groups, with dK/dV in shares
    "half_d64": ([700] * 130, None, 8, 2, 64),
    "half_d128": ([700] * 130, None, 8, 2, 128),
    "whole": ([2560] * 14, None, 8, 2, 128),
    "keys": ([16384, 16384], [8, 8], 16, 2, 128),
}


@pytest.mark.parametrize("name", sorted(PERSISTENT))
def test_persistent_units_against_masked_calls(name):
    """A workgroup that runs unit after unit leaves the results of workgroups that
    run one: some items of the list, each alone in a masked call of at most one
    workgroup a compute unit, bit for bit."""
    import torch
    require_gpu()
    lengths, sp, hq, hkv, D = PERSISTENT[name]
    wl = small_worklist(lengths, hq, hkv, D, sp=sp)
    g = torch.Generator(device="cuda")
    g.manual_seed(900 + len(name))
    scale = 1.0 / np.sqrt(D)
    sizes = (wl.q_elems(), wl.kv_elems(), wl.kv_elems(), wl.q_elems())
    q, k, v, do = (torch.randn(n, generator=g, device="cuda").to(torch.bfloat16) for n in sizes)

    def call(w):
        b = nsp.alloc_like_worklist(w, grad_dtype=torch.float32)
        for n in ("o", "lse", "dq", "dk", "dv"):
            b[n].fill_(float("nan"))
        nsp.nsp_varlen_attn_fwd(w, q, k, v, b["o"], b["lse"], scale)
        nsp.nsp_varlen_attn_bwd(w, q, k, v, b["o"], do, b["lse"], b["dq"], b["dk"], b["dv"], b["ws"], scale)
        torch.cuda.synchronize()
        return b

    full = call(wl)
    at = {n: np.concatenate([[0], np.cumsum(wl.lengths.astype(np.int64) * per)])
          for n, per in (("o", wl.hq * D), ("lse", wl.hq), ("dq", wl.hq * D), ("dk", wl.hkv * D), ("dv", wl.hkv * D))}
    for j in sorted({0, wl.n_items // 2, wl.n_items - 1}):
        mask = np.zeros(wl.n_items, np.uint8)
        mask[j] = 1
        one = call(wl.select(mask))
        for n, off in at.items():
            a, b = (t[n][off[j]:off[j + 1]] for t in (full, one))
            wide = torch.int16 if a.dtype == torch.bfloat16 else torch.int32
            assert bool(torch.isfinite(a).all()) and torch.equal(a.view(wide), b.view(wide)), (n, j)
