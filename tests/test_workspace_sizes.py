"""Workspaces of the sizes that earlier releases asked for are still enough, and
the allocation-free call still holds what it held.  No GPU: a call that passes
its argument and workspace checks then fails at its first launch
(WF_ERR_HIP), so the pointers are never followed."""
import ctypes

import pytest
import torch

PTR = 1 << 20  # aligned, never read
WORKSPACE, HIP = 3, 4


@pytest.fixture(scope="module")
def wf():
    if torch.cuda.is_available():
        pytest.skip("the calls would be launched")
    import paper_2606_00724_amd as m
    return m


def _p(wf, units, L, d, B, J, S, k, G, dtype, wavelet="haar", heads=1):
    return wf.make_params(batch=units // heads, heads=heads, ctx_len=L, head_dim=d, q_len=B,
                          levels=J, segments=S, budget=k, gen_len=G, dtype=dtype,
                          wavelet=wavelet)


def _call(wf, op, p, nbytes, rows=0, props=None):
    lib, P, f = wf.library(), ctypes.byref(p), PTR
    g = f if p.gen_len else None
    if op == "skim":
        return lib.wf_skim_score(P, f, f, f, f, f, nbytes, None)
    if op == "scan":
        return lib.wf_scan_select(P, f, f, f, None, f, f, nbytes, None)
    if op == "attn":
        rows = rows or (wf.effective_budget(p) + p.gen_len + p.ctx_len % (1 << p.levels))
        return lib.wf_sparse_attn(P, f, f, f, rows, f, f, nbytes, None)
    if op == "fused":
        return lib.wf_filter_attend(P, f, f, f, g, g, f, None, None, f, nbytes, None)
    if op == "cached":
        return lib.wf_filter_attend_cached(P, f, f, f, f, g, g, f, None, None, f, nbytes, None)
    if op == "shared":
        return lib.wf_filter_attend_shared(P, f, f, f, g, g, f, None, None, f, nbytes, None)
    if op == "noalloc":
        return lib.wf_filter_attend_noalloc(P, f, f, f, g, g, f, None, None, None)
    arr = (ctypes.c_float * p.levels)(*props)
    return lib.wf_filter_attend_recursive(P, arr, f, f, f, g, g, f, None, None, f, nbytes, None)


# rows of coarse logits whose length is no multiple of four
@pytest.mark.parametrize("op,args,nbytes", [
    ("skim", (8, 1024, 64, 128, 10, 1, 177, 0, "bf16"), 12288),
    ("skim", (152, 878, 64, 150, 6, 7, 293, 33, "bf16", "db2", 4), 1368320),
    ("skim", (90, 1024, 64, 256, 10, 1, 101, 5000, "f32", "haar", 2), 276480),
    ("skim", (360, 347, 64, 17, 1, 113, 24, 0, "f32", "haar", 8), 4382208),
    ("cached", (1, 86, 64, 100, 6, 1, 13, 0, "bf16", "db2"), 29952),
    ("cached", (2010, 245, 128, 16, 1, 30, 36, 33, "bf16", "db2"), 34894080),
    ("cached", (4, 8941, 64, 200, 3, 495, 436, 0, "bf16", "db2", 4), 5455872),
])
def test_unpadded_logits(wf, op, args, nbytes):
    assert _call(wf, op, _p(wf, *args), nbytes) == HIP
