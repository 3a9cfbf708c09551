"""Where the units of a pass run, which no output shows: timed.

* A persistent pass takes as long on one stream as on another.  Which XCD the
  first workgroup of a launch runs on depends on the stream's hardware queue, and
  the gangs of the unit queues have to stay on one XCD all the same: dK/dV of one
  head-sharded sequence of 594 key tiles took 11.7 ms against 10.1 on one of two
  streams while workgroups started with queue b % 8, and is within 1% with every
  unit from the own XCD's queue.
* A dK/dV pass of no more units than compute units lasts as long as its longest
  unit, wherever the queues put the units: twice as long for twice the tokens (and
  the start and end of a unit on top).  The one item of a masked call, 2048 and
  4096 tokens: 331 and 647 us, and 340 and 760 to 907 while a gang's units shared
  one XCD.
"""
import numpy as np
import pytest

from paper_2609_22755_amd import nsp
from paper_2609_22755_amd.workloads import small_worklist

from gpu_util import require_gpu

pytestmark = pytest.mark.gpu


def dkdv_times(lists, streams, reps=6):
    """Median dK/dV time (ms) of each (work list, stream), taken in turn."""
    import torch
    require_gpu()
    g = torch.Generator(device="cuda")
    g.manual_seed(91)
    calls = []
    for wl in lists:
        q, k, v, do = (torch.randn(n, generator=g, device="cuda").to(torch.bfloat16)
                       for n in (wl.q_elems(), wl.kv_elems(), wl.kv_elems(), wl.q_elems()))
        buf = nsp.alloc_like_worklist(wl)
        scale = 1.0 / np.sqrt(wl.head_dim)
        nsp.nsp_varlen_attn_fwd(wl, q, k, v, buf["o"], buf["lse"], scale)
        calls.append((wl, q, k, v, buf["o"], do, buf["lse"], buf["dq"], buf["dk"], buf["dv"], buf["ws"], scale))
    torch.cuda.synchronize()
    times = {(i, j): [] for i in range(len(lists)) for j in range(len(streams))}
    nsp.nsp_timing_enable(1)
    try:
        for rep in range(reps):
            for (i, j), t in times.items():
                nsp.nsp_timing_reset()
                nsp.nsp_varlen_attn_bwd(*calls[i], stream=streams[j])
                torch.cuda.synchronize()
                if rep > 0:                    # (rep 0: warm-up, and every stream has its queue)
                    t.append(nsp.nsp_timing_query("bwd_dkdv")[1])
    finally:
        nsp.nsp_timing_enable(0)
    med = {key: float(np.median(t)) for key, t in times.items()}
    print(f"[placement] dK/dV ms: {med}", flush=True)
    return med


def test_persistent_pass_is_as_fast_on_every_stream():
    import torch
    require_gpu()
    t = dkdv_times([small_worklist([594 * 128], 32, 4, 128, sp=[8])],
                   [torch.cuda.current_stream(), torch.cuda.Stream()])
    assert max(t.values()) <= 1.08 * min(t.values())


def test_few_units_run_at_once():
    import torch
    require_gpu()
    # (beside an item that makes the list too long for shares)
    lists = [small_worklist([L, 65536], 32, 4, 128).select([1, 0]) for L in (2048, 4096)]
    t = dkdv_times(lists, [torch.cuda.current_stream()])
    assert t[1, 0] <= 2.1 * t[0, 0]
