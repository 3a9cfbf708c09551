"""The split dK/dV pass: lists of few or long key tiles, whose steps are cut
into one share per compute unit and whose partial sums a second pass adds.

On the CPU the cuts are checked against brute force on random lists
(tests/native/split_checks.cpp).  On the GPU, at the sizes where a piece can go
wrong (pieces that start and end inside a query tile's heads, ragged ends, an
odd number of key tiles, one query head a KV head, a KV head with none, both
head widths, lists small enough for one launch with dQ), against the float64
oracle and against the whole tiles, which the same items run in a list of more
than 512 key tiles, the most that shares go up to (the others masked out): float32 sums of at most 2^16 terms in another order, whose relative difference
is bounded by about sqrt(2^16) * 2^-24 = 1.5e-5 for sums without cancellation
(P and dS themselves are computed alike, bit for bit).
"""
import dataclasses
import os
import shutil
import subprocess

import numpy as np
import pytest

from paper_2609_22755_amd import nsp
from paper_2609_22755_amd.workloads import draw_attention_inputs, make_config, small_worklist

from gpu_util import GRAD_REL_L2, oracle_full, rel_l2, report, require_gpu, run_attention, to_np

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
ROCM = "/opt/rocm"
SUM_REL = 1.5e-5


def padded(wl):
    """The work list with more than 512 one-token key tiles behind it, masked out."""
    k = 512 // wl.hkv_total + 1
    return dataclasses.replace(
        wl, lengths=np.concatenate([wl.lengths, np.ones(k, np.int32)]), sp=np.concatenate([wl.sp, np.ones(k, np.int32)]),
        q_heads=np.concatenate([wl.q_heads, np.tile([[0, wl.hq_total]], (k, 1))]),
        kv_heads=np.concatenate([wl.kv_heads, np.tile([[0, wl.hkv_total]], (k, 1))]),
        item_mask=np.concatenate([np.ones(wl.n_items, np.uint8), np.zeros(k, np.uint8)]))


def _lone_kv_head():
    """Query heads 0..3 of 8 use KV head 0; KV head 1 is held without any."""
    wl = small_worklist([1500], 8, 2, 128)
    return dataclasses.replace(wl, q_heads=np.array([[0, 4]], dtype=np.int32))


CASES = {
    "one_512": lambda: small_worklist([512], 32, 4, 128),
    "node_odd_tiles": lambda: small_worklist([1160], 32, 4, 128, sp=[8], rank=[3]),
    "mixed": lambda: small_worklist([700, 129, 1, 300, 2048, 0, 64], 32, 4, 128, sp=[2, 1, 1, 8, 4, 1, 1],
                                    rank=[1, 0, 0, 6, 3, 0, 0]),
    "mha": lambda: small_worklist([2999, 65], 2, 2, 128),
    "d64": lambda: small_worklist([2049, 500], 8, 2, 64),
    "lone_kv_head": _lone_kv_head,
    # small lists: dQ units in the same launch, with tiles cut and whole
    "small_mixed": lambda: small_worklist([200, 64, 33, 0, 1, 257], 32, 4, 128, sp=[2, 1, 1, 1, 1, 1],
                                          rank=[1, 0, 0, 0, 0, 0]),
    "small_d64": lambda: small_worklist([64, 129, 256, 511], 8, 2, 64),
    "small_whole": lambda: small_worklist([17, 31], 4, 2, 128),
}


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_split_cuts_on_random_lists(tmp_path):
    if not os.path.exists(os.path.join(ROCM, "include", "hip", "hip_runtime.h")):
        pytest.skip("HIP headers not available")
    csrc, native = os.path.join(ROOT, "paper_2609_22755_amd", "csrc"), os.path.join(ROOT, "tests", "native")
    exe = str(tmp_path / "split_checks")
    cmd = ["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-Wno-unknown-pragmas", "-I", csrc,
           "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROCM, "include"),
           os.path.join(native, "split_checks.cpp"), os.path.join(native, "launch_stubs.cpp"), "-o", exe,
           "-L", os.path.join(ROCM, "lib"), "-lamdhip64", f"-Wl,-rpath,{os.path.join(ROCM, 'lib')}"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    # the shares whose forward and dQ queues are checked for balance: the two of the
    # full-size tests, and each SP level's item-masked call of the long-tail one
    lists = tmp_path / "lists.txt"
    with open(lists, "w") as f:
        for name in ("longtail_4level", "maxctx_relayout"):
            wl = make_config(name).wl
            levels = sorted(set(int(x) for x in wl.sp)) if name == "longtail_4level" else []
            for sp in [0] + levels:
                f.write(f"{name}_sp{sp} {wl.hq_total} {wl.hkv_total} {wl.head_dim} {wl.n_items}\n")
                for j in range(wl.n_items):
                    f.write(" ".join(str(int(x)) for x in (wl.lengths[j], *wl.q_heads[j], *wl.kv_heads[j],
                                                           sp in (0, int(wl.sp[j])))) + "\n")
    r = subprocess.run([exe, str(lists)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and "split checks ok" in r.stdout, r.stdout + r.stderr


@pytest.mark.gpu
@pytest.mark.parametrize("name", sorted(CASES))
def test_split_gradients(name):
    import torch
    require_gpu()
    wl = CASES[name]()
    inp = draw_attention_inputs(wl, 300 + len(name))
    scale = 1.0 / np.sqrt(wl.head_dim)
    ref = oracle_full(wl, *inp, scale)
    g32 = run_attention(wl, *inp, scale, g_dtype=torch.float32)
    g16 = run_attention(wl, *inp, scale)
    q, k, v, do = (nsp.to_device_bf16(x) for x in inp)

    def again(call, wl_, x, ws=None):
        out = [torch.full((n,), float("nan"), dtype=torch.float32, device="cuda")
               for n in (wl_.q_elems(), wl_.kv_elems(), wl_.kv_elems())]
        args = (wl_, *x[:3], x[3], x[4], x[5], *out)
        call(*args, *(() if ws is None else (ws,)), scale)
        torch.cuda.synchronize()
        return out

    own = (q, k, v, g32["o"], do, g32["lse"])
    big = padded(wl)
    wide = [torch.cat([t, torch.zeros(n - t.numel(), dtype=t.dtype, device="cuda")]) for t, n in
            zip(own, (big.q_elems(), big.kv_elems(), big.kv_elems(), big.q_elems(), big.q_elems(), big.lse_elems()))]
    whole = again(nsp.nsp_varlen_attn_bwd, big, wide,
                  torch.empty(nsp.nsp_varlen_attn_bwd_workspace(big), dtype=torch.uint8, device="cuda"))
    errs = {}
    for n, w in zip(("dq", "dk", "dv"), whole):
        errs[n] = rel_l2(to_np(g16[n]), ref[n])
        errs[n + "32"] = rel_l2(to_np(g32[n]), ref[n])
        errs[n + "_whole"] = rel_l2(to_np(g32[n]), to_np(w)[:g32[n].numel()])
    report(f"split {name}", **errs)
    for n in ("dq", "dk", "dv"):
        assert errs[n] <= GRAD_REL_L2 and errs[n + "32"] <= GRAD_REL_L2 and errs[n + "_whole"] <= SUM_REL, n
    # the allocation-free call runs the same pieces
    for n, t in zip(("dq", "dk", "dv"), again(nsp.nsp_varlen_attn_bwd_noalloc, wl, own)):
        assert torch.equal(t.view(torch.int32), g32[n].view(torch.int32)), n
    # and so does a masked call, for its items alone
    mask = (np.arange(wl.n_items) % 2 == (wl.n_items - 1) % 2).astype(np.uint8)
    got = again(nsp.nsp_varlen_attn_bwd, wl.select(mask), own, g32["ws"])
    for n, t, per in zip(("dq", "dk", "dv"), got, (wl.hq, wl.hkv, wl.hkv)):
        at = np.concatenate([[0], np.cumsum(wl.lengths.astype(np.int64) * per * wl.head_dim)])
        for j in range(wl.n_items):
            a, b = t[at[j]:at[j + 1]], g32[n][at[j]:at[j + 1]]
            assert torch.equal(a.view(torch.int32), b.view(torch.int32)) if mask[j] else bool(torch.isnan(a).all()), (n, j)
