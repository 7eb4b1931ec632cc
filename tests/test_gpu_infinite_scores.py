"""Keys whose score is -inf for every query (an infinite channel): weight 0 in
the scan and in the attention, wherever they stand in a range, a chunk or a
block of 16 rows, as the softmax over the other rows gives it."""
import pytest
import torch

from parity import O_TOL, SEL_REL

pytestmark = pytest.mark.gpu


def rows_of(n, spans):
    bad = torch.zeros(n, dtype=torch.bool)
    for a, b in spans:
        bad[a:b] = True
    return bad.cuda()


def inputs(units, rows, n, d, dtype, bad):
    gen = torch.Generator(device="cuda").manual_seed(rows + n)
    Q = torch.randn(1, units, rows, d, generator=gen, device="cuda")
    K = torch.randn(1, units, n, d, generator=gen, device="cuda")
    V = torch.randn(1, units, n, d, generator=gen, device="cuda")
    Q[..., 0] = Q[..., 0].abs() + 0.5
    Q, K, V = (x.to(dtype) for x in (Q, K, V))
    K[:, :, bad, 0] = float("-inf")
    return Q, K, V


# whole blocks of 16 rows, the first rows, the last, every other row
SPANS = [[(16, 32)], [(0, 16)], [(0, 1), (63, 130)], [(i, i + 1) for i in range(0, 200, 2)]]


@pytest.mark.parametrize("spans", SPANS, ids=["block", "first", "ends", "alternate"])
@pytest.mark.parametrize("d,B", [(64, 16), (128, 50), (64, 130)])
def test_fp32_attention(spans, d, B):
    import paper_2606_00724_amd as wf
    units, n = 3, 200
    p = wf.make_params(batch=1, heads=units, ctx_len=4096, head_dim=d, q_len=B, levels=3,
                       segments=512, budget=n, dtype="f32")
    bad = rows_of(n, spans)
    Q, K, V = inputs(units, B, n, d, torch.float32, bad)
    O = torch.empty_like(Q)
    wf.wf_sparse_attn(p, Q, K, V, n, O, wf.alloc_workspace(p, wf.OP_ATTN, Q.device))
    torch.cuda.synchronize()
    Kd, Vd = K[0][:, ~bad].double(), V[0][:, ~bad].double()
    ref = torch.softmax(Q[0].double() @ Kd.transpose(1, 2).contiguous() / d ** 0.5, -1) @ Vd
    assert (O[0] - ref).abs().max().item() <= O_TOL["f32"]


@pytest.mark.parametrize("spans", SPANS, ids=["block", "first", "ends", "alternate"])
@pytest.mark.parametrize("dtype,d,B", [("f32", 64, 16), ("f32", 128, 70), ("bf16", 128, 33),
                                       ("bf16", 64, 100)])
def test_scan(spans, dtype, d, B):
    import paper_2606_00724_amd as wf
    units, S, J = 600, 50, 3  # one range a unit, several chunks
    n = S << J
    p = wf.make_params(batch=1, heads=units, ctx_len=n, head_dim=d, q_len=B, levels=J, segments=S,
                       budget=n // 2, dtype=dtype)
    bad = rows_of(n, spans)
    Q, K, _ = inputs(units, B, n, d, wf.torch_dtype(p), bad)
    seg = torch.arange(S, dtype=torch.int32, device="cuda").repeat(units, 1).contiguous()
    W = torch.empty((units, n), device="cuda")
    tok = torch.empty((units, n // 2), dtype=torch.int32, device="cuda")
    wf.wf_scan_select(p, Q, K, seg, W, tok, wf.alloc_workspace(p, wf.OP_SCAN, Q.device))
    torch.cuda.synchronize()
    pick = [0, 299, 599]
    s = Q[0][pick].double() @ K[0][pick][:, ~bad].double().transpose(1, 2).contiguous() / d ** 0.5
    ref = torch.softmax(s, -1).sum(1)
    assert (W[:, bad] == 0).all()
    assert ((W[pick][:, ~bad] - ref).abs() / ref).max().item() <= SEL_REL


# rows that fill no last block of 16 or chunk of 64, in one split and in several;
# the row parts of two (50 rows) and four waves (16)
@pytest.mark.parametrize("units,n", [(3, 1), (3, 17), (3, 200), (300, 95), (600, 4099)])
@pytest.mark.parametrize("d,B", [(64, 16), (128, 50)])
def test_fp32_infinite_value_in_the_last_row(units, n, d, B):
    """Channels of V that are infinite in the last row: infinite there for every
    query, as each weight is positive, and the other channels as without them."""
    import paper_2606_00724_amd as wf
    p = wf.make_params(batch=1, heads=units, ctx_len=8192, head_dim=d, q_len=B, levels=1,
                       segments=4096, budget=n, dtype="f32")
    Q, K, V = inputs(units, B, n, d, torch.float32, rows_of(n, []))
    ref = torch.softmax(Q[0].double() @ K[0].double().transpose(1, 2).contiguous() / d ** 0.5,
                        -1) @ V[0].double()
    V[:, :, -1, 0], V[:, :, -1, d - 1] = float("inf"), float("-inf")
    O = torch.empty_like(Q)
    wf.wf_sparse_attn(p, Q, K, V, n, O, wf.alloc_workspace(p, wf.OP_ATTN, Q.device))
    torch.cuda.synchronize()
    assert (O[..., 0] == float("inf")).all() and (O[..., d - 1] == float("-inf")).all()
    assert (O[0] - ref)[..., 1:d - 1].abs().max().item() <= O_TOL["f32"]
