"""fp32 keys and large scores: the products are exact in fp32 (a scale of 1/8 and
short integers), so the weights are those of the exact scores, however large the
scores are beside their differences."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def inputs(units, B, n, d, seed):
    """Scores of 2048 + multiples of 1/32 (1/sqrt(128) is no power of two:
    d = 64 only), differing by at most 8 within a query."""
    gen = torch.Generator(device="cuda").manual_seed(seed)

    def ints(*shape, lo, hi):
        return torch.randint(lo, hi, shape, generator=gen, device="cuda").float()
    Q = torch.zeros(1, units, B, d, device="cuda")
    K = torch.zeros(1, units, n, d, device="cuda")
    Q[..., 0], K[..., 0] = 128.0, 128.0
    Q[..., 1:17] = ints(1, units, B, 16, lo=-1, hi=2)
    K[..., 1:17] = ints(1, units, n, 16, lo=-8, hi=9) / 4
    V = torch.randn(1, units, n, d, generator=gen, device="cuda")
    return Q, K, V


# exponents: 12 log2(e) rounded relatively by 2^-24 twice (the constant, the
# scaled constant) and the exponential's 2^-22, each of a sum of up to 1000
# terms and of its merges rounded to 2^-24: 4e-6 of weights that sum to 1
REL = 4e-6


@pytest.mark.parametrize("units,n,B", [(1, 16, 1), (2, 1000, 17), (3, 300, 64), (40, 777, 130)])
def test_attention(units, n, B):
    import paper_2606_00724_amd as wf
    d = 64
    p = wf.make_params(batch=1, heads=units, ctx_len=4096, head_dim=d, q_len=B, levels=3,
                       segments=512, budget=n, dtype="f32")
    Q, K, V = inputs(units, B, n, d, 3)
    O = torch.empty_like(Q)
    wf.wf_sparse_attn(p, Q, K, V, n, O, wf.alloc_workspace(p, wf.OP_ATTN, Q.device))
    torch.cuda.synchronize()
    s = Q[0].double() @ K[0].double().transpose(1, 2).contiguous() / 8
    assert s.max() - s.min() <= 20 and s.min() > 2000
    w = torch.softmax(s, -1)
    bound = REL * (w @ V[0].double().abs())
    err = (O[0] - w @ V[0].double()).abs()
    print("worst error over the bound", (err / bound).max().item(), flush=True)
    assert (err <= bound).all()


@pytest.mark.parametrize("units,S,B", [(1, 8, 1), (2, 100, 17), (3, 40, 64), (300, 30, 130)])
def test_scan(units, S, B):
    import paper_2606_00724_amd as wf
    d, J = 64, 3
    n = S << J
    p = wf.make_params(batch=1, heads=units, ctx_len=n, head_dim=d, q_len=B, levels=J, segments=S,
                       budget=n // 2, dtype="f32")
    Q, K, _ = inputs(units, B, n, d, 4)
    seg = torch.arange(S, dtype=torch.int32, device="cuda").repeat(units, 1).contiguous()
    W = torch.empty((units, n), device="cuda")
    tok = torch.empty((units, n // 2), dtype=torch.int32, device="cuda")
    wf.wf_scan_select(p, Q, K, seg, W, tok, wf.alloc_workspace(p, wf.OP_SCAN, Q.device))
    torch.cuda.synchronize()
    ref = torch.softmax(Q[0].double() @ K[0].double().transpose(1, 2).contiguous() / 8, -1).sum(1)
    rel = ((W - ref).abs() / ref).max().item()
    print("worst relative error over the bound", rel / REL, flush=True)
    assert rel <= REL
