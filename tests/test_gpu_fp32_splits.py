"""fp32 splits and ranges: with the finer workspace and with the smaller one that
earlier releases asked for, and splits of more rows than their token ids fit
the LDS, against torch in float64."""
import pytest
import torch

from parity import O_TOL

pytestmark = pytest.mark.gpu

TOL = O_TOL["f32"]


@pytest.fixture(scope="module")
def wf():
    import paper_2606_00724_amd as m
    return m


def up256(x):
    return (x + 255) & ~255


def attend64(q, k, v):
    s = q.double() @ k.double().T / q.shape[-1] ** 0.5
    return torch.softmax(s, dim=-1) @ v.double()


# rows: one chunk, a chunk and one row, several chunks, several splits
@pytest.mark.parametrize("units,rows,d,B", [
    (1, 40, 64, 17), (1, 65, 128, 100), (3, 200, 64, 45), (2, 200, 128, 160), (5, 1000, 128, 33),
    (129, 1000, 64, 8), (265, 130, 64, 64), (600, 20, 64, 1)])
@pytest.mark.parametrize("former", [False, True])
def test_staged_attention(wf, units, rows, d, B, former):
    p = wf.make_params(batch=1, heads=units, ctx_len=4096, head_dim=d, q_len=B, levels=3,
                       segments=512, budget=rows, dtype="f32")
    print(f"attention units={units} rows={rows} d={d} B={B} former={former}", flush=True)
    torch.manual_seed(rows)
    Q = torch.randn(1, units, B, d, device="cuda")
    K, V = (torch.randn(1, units, rows, d, device="cuda") for _ in range(2))
    nbytes = wf.workspace_bytes(p, wf.OP_ATTN)
    if former:  # splits of whole 128-row chunks, about 512 in all
        chunks = (rows + 127) // 128
        splits = min(chunks, max(1, (512 + units - 1) // units))
        splits = -(-chunks // -(-chunks // splits))
        nbytes = up256(units * splits * B * d * 4) + up256(units * splits * 2 * B * 4)
    O = torch.full_like(Q, float("nan"))
    ws = torch.full((nbytes,), 255, dtype=torch.uint8, device="cuda")
    wf.wf_sparse_attn(p, Q, K, V, rows, O, ws)
    torch.cuda.synchronize()
    ref = torch.stack([attend64(Q[0, u], K[0, u], V[0, u]) for u in range(units)])
    assert (O[0] - ref).abs().max().item() <= TOL


@pytest.mark.parametrize("units,S,J,d,B", [
    (1, 8, 3, 64, 17), (2, 33, 2, 128, 100), (4, 49, 5, 128, 160), (129, 32, 4, 64, 32),
    (266, 16, 3, 128, 17)])
@pytest.mark.parametrize("former", [False, True])
def test_staged_scan(wf, units, S, J, d, B, former):
    L = 2 * S << J
    p = wf.make_params(batch=1, heads=units, ctx_len=L, head_dim=d, q_len=B, levels=J,
                       segments=S, budget=(S << J) // 2, dtype="f32")
    print(f"scan units={units} S={S} J={J} d={d} B={B} former={former}", flush=True)
    torch.manual_seed(S)
    Q, K = (torch.randn(1, units, n, d, device="cuda") for n in (B, L))
    seg = (2 * torch.arange(S, dtype=torch.int32, device="cuda")).repeat(units, 1).contiguous()
    P, nbytes = S << J, wf.workspace_bytes(p, wf.OP_SCAN)
    if former:  # ranges of 1 to 8 chunks of 128 positions, about 1024 in all
        chunks = (P + 127) // 128
        cpw = max(1, min(8, units * chunks // 1024))
        nbytes = up256(units * -(-chunks // cpw) * 2 * B * 4) + up256(units * P * 4)
    W = torch.full((units, P), float("nan"), device="cuda")
    tok = torch.empty((units, P // 2), dtype=torch.int32, device="cuda")
    wf.wf_scan_select(p, Q, K, seg, W, tok, torch.empty(nbytes, dtype=torch.uint8, device="cuda"))
    torch.cuda.synchronize()
    rows = ((seg[0].long() << J)[:, None] + torch.arange(1 << J, device="cuda")).reshape(-1)
    for u in {0, units // 2, units - 1}:
        s = Q[0, u].double() @ K[0, u, rows].double().T / d ** 0.5
        ref = torch.softmax(s, dim=-1).sum(0)
        # a logit of magnitude below 8 carries d rounded products: d 2^-24 8
        # relative in its weight at most
        assert ((W[u] - ref).abs() / ref).max().item() <= 8 * d * 2.0 ** -24
        assert (tok[u][1:] > tok[u][:-1]).all()


def test_splits_of_more_rows_than_ids_in_lds(wf):
    """1100 units, a budget of 9000 tokens and a tail: at most two splits a unit,
    of more rows than the 4096 token ids that wait in LDS at once."""
    U, L, d, B, G = 1100, 9403, 64, 5, 33
    p = wf.make_params(batch=1, heads=U, ctx_len=L, head_dim=d, q_len=B, levels=3, segments=1150,
                       budget=9000, gen_len=G, dtype="f32")
    assert "scan_select" in wf.fused_kernel_names(p)
    torch.manual_seed(7)
    Q, K, V, Kg, Vg = (torch.randn(1, U, n, d, device="cuda") for n in (B, L, L, G, G))
    print("fused 1100 x 9000 rows", flush=True)
    O, tok, _ = wf.filter_attend(p, Q, K, V, Kg, Vg, want_indices=True)
    torch.cuda.synchronize()
    for u in (0, 1, 517, 1099):
        t = tok.reshape(U, -1)[u].long()
        assert t.numel() == 9000 and (t[1:] > t[:-1]).all()
        rows = torch.cat([t, torch.arange(L // 8 * 8, L, device="cuda")])
        ref = attend64(Q[0, u], torch.cat([K[0, u, rows], Kg[0, u]]),
                       torch.cat([V[0, u, rows], Vg[0, u]]))
        assert (O[0, u] - ref).abs().max().item() <= TOL


def least_bytes(wf, run, need):
    """the fewest bytes (a multiple of 256) that run(bytes) takes"""
    lo, hi = 0, need // 256
    while lo < hi:
        mid = (lo + hi) // 2
        try:
            run(mid * 256)
            hi = mid
        except wf.WfError as e:
            assert e.status == 3, e
            lo = mid + 1
    return hi * 256


@pytest.mark.parametrize("units,L,d,B,J,S,k,G", [
    (2, 1024, 64, 32, 3, 32, 128, 0), (7, 1810, 128, 64, 4, 113, 806, 0),
    (13, 5184, 128, 8, 5, 16, 197, 33), (129, 520, 64, 17, 2, 40, 100, 300)])
@pytest.mark.parametrize("call", ["fused", "cached", "shared"])
def test_whole_step_with_less_workspace(wf, call, units, L, d, B, J, S, k, G):
    p = wf.make_params(batch=1, heads=units, ctx_len=L, head_dim=d, q_len=B, levels=J, segments=S,
                       budget=k, gen_len=G, dtype="f32")
    torch.manual_seed(11)
    Q, K, V = (torch.randn(1, units, n, d, device="cuda") for n in (B, L, L))
    Kg, Vg = (torch.randn(1, units, G, d, device="cuda") if G else None for _ in range(2))
    op = {"fused": wf.OP_FUSED, "cached": wf.OP_CACHED, "shared": wf.OP_SHARED}[call]
    need = wf.workspace_bytes(p, op)
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    A = wf.dwt_approx(p, K)
    tok = torch.empty((units if call != "shared" else 1, wf.effective_budget(p)),
                      dtype=torch.int32, device="cuda")

    def run(nbytes):
        O = torch.full_like(Q, float("nan"))
        ws.fill_(255)
        if call == "fused":
            wf.wf_filter_attend(p, Q, K, V, Kg, Vg, O, tok, None, ws[:nbytes])
        elif call == "cached":
            wf.wf_filter_attend_cached(p, Q, A, K, V, Kg, Vg, O, tok, None, ws[:nbytes])
        else:
            wf.wf_filter_attend_shared(p, Q, K, V, Kg, Vg, O, tok, None, ws[:nbytes])
        torch.cuda.synchronize()
        return O, tok.clone()
    O1, t1 = run(need)
    least = least_bytes(wf, run, need)
    print(f"{call} units={units}: {need} bytes asked for, {least} enough", flush=True)
    O2, t2 = run(least)
    assert (t1 != t2).sum() <= 2 * units  # a near-tie may go the other way
    same = (t1 == t2).all(1)
    if call != "shared":
        assert same.sum() >= units - 2
        O1, O2 = O1[0, same], O2[0, same]
    if same.any():
        assert (O1 - O2).abs().max().item() <= TOL
