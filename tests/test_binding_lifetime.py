"""The binding keeps a work list's host arrays alive for the whole call: lists
of several hundred items, whose arrays the allocator hands out again at once
when they are freed (short ones often keep their contents by luck)."""
import ctypes

import numpy as np
import pytest

from paper_2609_22755_amd import nsp
from paper_2609_22755_amd.workloads import small_worklist


@pytest.mark.parametrize("n_items", [3, 300, 2000])
def test_workspace_query_of_long_lists(n_items):
    wl = small_worklist([1 + j % 7 for j in range(n_items)], 8, 2, 64)
    rows = -(-4 * wl.lse_elems() // 256) * 256          # a float32 a row, 256-byte aligned
    assert nsp.nsp_varlen_attn_bwd_workspace(wl) == 2 * rows + 256 + 512 * 1024 * 64


@pytest.mark.parametrize("call", ["pack", "unpack"])
def test_relayout_passes_the_list_it_was_given(monkeypatch, call):
    wl = small_worklist([2 * (1 + j % 7) for j in range(2000)], 8, 2, 64, sp=[2] * 2000)
    lib = nsp.load_library()
    seen = {}

    class Lib:
        def __getattr__(self, name):
            def f(ref, *args):
                c = ctypes.cast(ref, ctypes.POINTER(nsp.CWorkList)).contents
                seen["cu"] = np.ctypeslib.as_array(c.cu_seqlens, (c.n_items + 1,)).copy()
                return nsp.NSP_OK
            return f
    monkeypatch.setattr(nsp, "load_library", lambda: Lib())
    import torch
    t = torch.zeros(16, dtype=torch.bfloat16)
    if call == "pack":
        nsp.nsp_ulysses_pack(wl, nsp.NSP_KIND_Q, t, t, stream=0)
    else:
        nsp.nsp_ulysses_unpack(wl, nsp.NSP_KIND_Q, nsp.NSP_UNPACK_SELECT, t, t, stream=0)
    assert np.array_equal(seen["cu"], wl.cu_seqlens) and lib is not None
