"""Dispatch edges of the coefficient-tile path and its rings: every unit of the
fused, cached and shared calls against the fp64 oracle (the tolerances of
parity.py)."""
import pytest

import synth
from test_gpu_random_shapes import _check_case

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def wf():
    import paper_2606_00724_amd as m
    return m


def _w(name, **kw):
    base = dict(batch=1, heads=4, head_dim=128, q_len=32, dtype="bf16", wavelet="haar",
                boundary="symmetric", gen_len=0, needles=1, seed=41)
    base.update(kw)
    return synth.small_variant(synth.WORKLOADS["tiny"], name=name, **base)


# W over all CUs and the selections in their consumers from 1024 coefficients
# in all: just below and at the line, past 64 query rows, coefficient counts
# that are no multiple of four
WIDE = [
    _w("w1023", heads=3, ctx_len=341 * 8, levels=3, segments=40, budget=300, q_len=65),
    _w("w1024", heads=4, ctx_len=256 * 8, levels=3, segments=40, budget=300, q_len=65),
    _w("w_b128", heads=4, ctx_len=4 * 513 + 3, levels=2, segments=99, budget=150, q_len=128,
       gen_len=9),
    _w("w_b256", heads=2, ctx_len=64 * 514, levels=6, segments=3, budget=100, q_len=256,
       head_dim=64),
    _w("w_pad1", heads=4, ctx_len=4 * 259 + 1, levels=2, segments=259, budget=1036, q_len=17),
    _w("w_db2", heads=5, ctx_len=16 * 301, levels=4, segments=20, budget=90, q_len=48,
       wavelet="db2", boundary="periodic"),
    _w("w_j7", heads=8, ctx_len=128 * 130, levels=7, segments=9, budget=200, q_len=64),
]


@pytest.mark.parametrize("w", WIDE, ids=lambda w: w.name)
def test_wide_route(wf, w):
    names = wf.fused_kernel_names(wf.params_for(w))
    wide = w.name != "w1023"
    assert names[1] == ("skim_weights" if wide else "skim_select"), names
    _check_case(wf, w, w.name, "wide", cached=True)


# fp32 keys through the rings: query blocks shared by two waves (1 to 16 of
# them), one chunk, a chunk and one row, several chunks, both head sizes, a
# remainder and a tail; below 1024 coefficients the select kernels
F32 = [
    _w("f_b1", dtype="f32", heads=2, ctx_len=1024, levels=3, segments=8, budget=64, q_len=1),
    _w("f_b16", dtype="f32", heads=2, ctx_len=1029, levels=3, segments=9, budget=65, q_len=16,
       head_dim=64, gen_len=3),
    _w("f_b33", dtype="f32", heads=4, ctx_len=8 * 300 + 5, levels=3, segments=60, budget=257,
       q_len=33, gen_len=40),
    _w("f_b64", dtype="f32", heads=8, ctx_len=4096, levels=4, segments=100, budget=700, q_len=64),
    _w("f_b100", dtype="f32", heads=6, ctx_len=4 * 257, levels=2, segments=64, budget=100,
       q_len=100, head_dim=64),
    _w("f_b160", dtype="f32", heads=4, ctx_len=4 * 300, levels=2, segments=64, budget=100,
       q_len=160),
    _w("f_long", dtype="f32", heads=1, ctx_len=32 * 1030, levels=5, segments=400, budget=5000,
       q_len=20, wavelet="db2"),
]


@pytest.mark.parametrize("w", F32, ids=lambda w: w.name)
def test_fp32_rings(wf, w):
    _check_case(wf, w, w.name, "fp32", cached=True)


@pytest.mark.parametrize("rows,d,taken", [(169, 128, True), (170, 128, False), (176, 128, False),
                                          (256, 64, True)])
def test_fp32_query_rows_keep_their_limit(wf, rows, d, taken):
    """The two-pass scan takes up to 169 fp32 rows of 128 channels (all 256 of 64):
    one more is an error of the scan's launch."""
    import torch
    p = wf.make_params(batch=1, heads=1, ctx_len=1024, head_dim=d, q_len=rows, levels=3,
                       segments=8, budget=32, dtype="f32")
    x = torch.randn(1, 1, 1024, d, generator=torch.Generator().manual_seed(1)).cuda()
    q = x[:, :, :rows].contiguous()
    if taken:
        O = wf.filter_attend(p, q, x, x)
        torch.cuda.synchronize()
        assert torch.isfinite(O).all()
    else:
        with pytest.raises(wf.WfError, match="scan_stats") as e:
            wf.filter_attend(p, q, x, x)
        assert e.value.status_name == "WF_ERR_HIP"
        torch.cuda.synchronize()


# the selections past the register reach of 8192 scores (32 a thread up to
# 16384, then from LDS or memory), on the token-level path and the general one
POOL = [
    _w("p8192", heads=1, ctx_len=16384, levels=3, segments=1024, budget=4000),
    _w("p8200", heads=1, ctx_len=16384, levels=3, segments=1025, budget=4001),
    _w("p16384", heads=1, ctx_len=32768, levels=5, segments=512, budget=9000, gen_len=5),
    _w("p16416", heads=1, ctx_len=32768, levels=5, segments=513, budget=3000),
    _w("p27136", heads=1, ctx_len=27136 + 17, levels=6, segments=424, budget=20000, q_len=16),
]


@pytest.mark.parametrize("w", POOL, ids=lambda w: w.name)
def test_large_pools(wf, w):
    _check_case(wf, w, w.name, "pool", cached=True)


@pytest.mark.parametrize("dtype,levels", [("bf16", 3), ("bf16", 2), ("f32", 2)])
def test_equal_scores_need_no_pass(wf, dtype, levels):
    """Equal keys: no two scores differ, the lowest positions are taken."""
    import torch
    p = wf.make_params(batch=1, heads=20, ctx_len=1024, head_dim=128, q_len=32, levels=levels,
                       segments=40, budget=70, dtype=dtype)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    K = torch.ones(1, 20, 1024, 128, dtype=dt, device="cuda")
    Q = torch.full((1, 20, 32, 128), 0.25, dtype=dt, device="cuda")
    for _ in range(3):
        O, tok, seg = wf.filter_attend(p, Q, K, K, want_indices=True)
        torch.cuda.synchronize()
        assert (seg.cpu() == torch.arange(40, dtype=torch.int32)).all()
        assert (tok.cpu() == torch.arange(70, dtype=torch.int32)).all()


# unit counts that do not divide the CUs.  The r*_ cases of 16384 keys and r40_f32p
# take fewer, longer ranges in every kernel of their sequence (test_plan_limits.py
# asserts it); the others the counts of other remainders, and of more units than CUs
RANGES = [
    _w("r28_token", heads=28, ctx_len=16384 + 5, levels=4, segments=720, budget=5760, head_dim=64,
       q_len=17),
    _w("r28_held32", heads=28, ctx_len=16384, levels=5, segments=360, budget=5760, head_dim=64,
       q_len=17),
    _w("r28_db2p", heads=28, ctx_len=16384, levels=6, segments=180, budget=5760, head_dim=64,
       q_len=17, wavelet="db2"),
    _w("r28_pool", heads=28, ctx_len=16384, levels=2, segments=2880, budget=5760, head_dim=64,
       q_len=17),
    _w("r40_f32p", heads=40, ctx_len=8 * 640 + 3, levels=3, segments=320, budget=2560,
       head_dim=64, q_len=17, dtype="f32"),
    _w("r28_held", heads=28, ctx_len=32 * 330 + 7, levels=5, segments=30, budget=500),
    _w("r28_two", heads=28, ctx_len=8 * 700, levels=3, segments=90, budget=500, head_dim=64),
    _w("r100", heads=100, ctx_len=16 * 130, levels=4, segments=20, budget=200, q_len=17),
    _w("r28_db2", heads=28, ctx_len=64 * 70, levels=6, segments=12, budget=300, wavelet="db2"),
    _w("r28_general", heads=28, ctx_len=4 * 900, levels=2, segments=200, budget=500, q_len=40),
    _w("r40_f32", heads=40, ctx_len=8 * 200, levels=3, segments=60, budget=300, dtype="f32"),
    _w("r300", heads=300, ctx_len=8 * 40, levels=3, segments=20, budget=100, q_len=8),
]


@pytest.mark.parametrize("w", RANGES, ids=lambda w: w.name)
def test_ranges_of_odd_unit_counts(wf, w):
    _check_case(wf, w, w.name, "ranges", cached=True)


@pytest.mark.parametrize("dtype,L,J,d", [("bf16", 65536, 2, 128), ("f32", 32768, 2, 128),
                                         ("bf16", 131072 + 3, 6, 64)])
def test_streamed_haar_tiles(wf, dtype, L, J, d):
    """Keys past 256 MiB off the token-level path: tiles read with the streaming
    policy.  W and the regions of a few units from the cached call on the same A_J,
    which has no such tiles."""
    import torch
    units, B = 18, 20
    S = (L >> J) // 9
    p = wf.make_params(batch=1, heads=units, ctx_len=L, head_dim=d, q_len=B, levels=J, segments=S,
                       budget=300, dtype=dtype)
    dt = wf.torch_dtype(p)
    assert units * L * d * dt.itemsize > 256 << 20
    assert wf.fused_kernel_names(p)[0] == "skim_tile"
    gen = torch.Generator(device="cuda").manual_seed(9)
    K = torch.randn(1, units, L, d, generator=gen, device="cuda").to(dt)
    Q = torch.randn(1, units, B, d, generator=gen, device="cuda").to(dt)
    n = (L >> J) << J
    A = wf.dwt_approx(p, K)
    for u in (0, 7, 17):
        ref = K[0, u, :n].double().reshape(n >> J, 1 << J, d).sum(1) * 2.0 ** (-J / 2)
        # 2^J rows of at most 6 added in fp32
        assert (A[0, u] - ref).abs().max().item() <= (1 << J) ** 1.5 * 6 * 2.0 ** -24
    O1, t1, s1 = wf.filter_attend(p, Q, K, K, want_indices=True)
    O2, t2, s2 = wf.filter_attend_cached(p, Q, A, K, K, want_indices=True)
    torch.cuda.synchronize()
    same = (s1.reshape(units, -1) == s2.reshape(units, -1)).all(1)
    same &= (t1.reshape(units, -1) == t2.reshape(units, -1)).all(1)
    assert same.sum() >= units - 2  # a near-tie may go the other way
    assert (O1[0, same] - O2[0, same]).abs().max().item() <= (2e-2 if dtype == "bf16" else 1e-4)


@pytest.mark.parametrize("dtype,d", [("f32", 64), ("f32", 128), ("bf16", 128)])
def test_streamed_pools_and_raised_references(wf, dtype, d):
    """Pools past 32 MiB (streamed in the statistics pass), several chunks a
    range, logits that grow along the pool: lanes raise their reference again and
    again past their first block."""
    import torch
    from parity import SEL_REL
    units, S, J, B = 40, 520, 3, 33
    n = S << J
    p = wf.make_params(batch=1, heads=units, ctx_len=n, head_dim=d, q_len=B, levels=J, segments=S,
                       budget=100, dtype=dtype)
    dt = wf.torch_dtype(p)
    assert units * n * d * dt.itemsize > 32 << 20
    gen = torch.Generator(device="cuda").manual_seed(10)
    K = torch.randn(1, units, n, d, generator=gen, device="cuda")
    Q = torch.randn(1, units, B, d, generator=gen, device="cuda")
    Q[..., 0] = d ** 0.5
    K[..., 0] = torch.arange(n, device="cuda") * 0.25  # natural units: 2 a chunk row of 8
    Q, K = Q.to(dt), K.to(dt)
    s = Q[0, 3].double() @ K[0, 3].double().T / d ** 0.5
    # a lane sees every 128th position at least: its logits grow by more than
    # the 16 log2 units that its reference may lag
    assert ((s[:, 128:] - s[:, :-128]) * 1.4427 > 16).all()
    seg = torch.arange(S, dtype=torch.int32, device="cuda").repeat(units, 1).contiguous()
    W = torch.empty((units, n), device="cuda")
    tok = torch.empty((units, 100), dtype=torch.int32, device="cuda")
    wf.wf_scan_select(p, Q, K, seg, W, tok, wf.alloc_workspace(p, wf.OP_SCAN, Q.device))
    torch.cuda.synchronize()
    for u in (0, 3, 39):
        s = Q[0, u].double() @ K[0, u].double().T / d ** 0.5
        ref = torch.softmax(s, -1).sum(0)
        big = ref > 1e-20  # smaller ones are below 2^-126 in some query's units
        assert ((W[u] - ref).abs() / ref)[big].max().item() <= SEL_REL
