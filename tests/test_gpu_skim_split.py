"""The staged skim where W and the selection are one kernel, two, or W takes the
kernel of a thread per four columns: scores and regions against torch in
float64."""
import pytest
import torch

from parity import check_scores, check_selection

pytestmark = pytest.mark.gpu


# (units, columns, rows): either side of each line of the dispatch (1024
# coefficients in all, 512 columns, eight units a row, 256 units, 4096 columns,
# 64 rows, a workgroup of 1024 columns per CU), unit counts that leave a part
# more than fit the CUs, columns that are no multiple of four
@pytest.mark.parametrize("units,columns,rows", [
    (1, 1023, 3), (2, 512, 1), (64, 512, 8), (63, 510, 8), (64, 516, 8), (256, 128, 32),
    (257, 130, 32), (48, 1024, 17), (96, 511, 16), (300, 66, 256), (5, 4096, 8),
    (64, 4096, 63), (64, 4096, 64), (64, 4099, 16), (37, 8196, 5), (1, 9000, 200)])
@pytest.mark.parametrize("dtype,d", [("f32", 64), ("bf16", 128)])
def test_staged_skim(units, columns, rows, dtype, d):
    import paper_2606_00724_amd as wf
    S = max(1, columns // 7)
    p = wf.make_params(batch=1, heads=units, ctx_len=2 * columns + 1, head_dim=d, q_len=rows,
                       levels=1, segments=S, budget=1, dtype=dtype)
    print(f"skim units={units} columns={columns} rows={rows} {dtype}", flush=True)
    torch.manual_seed(columns)
    Q = torch.randn(1, units, rows, d, device="cuda").to(wf.torch_dtype(p))
    A = torch.randn(1, units, columns, d, device="cuda")
    W = torch.full((units, columns), float("nan"), device="cuda")
    seg = torch.full((units, S), -1, dtype=torch.int32, device="cuda")
    ws = torch.full((wf.workspace_bytes(p, wf.OP_SKIM),), 255, dtype=torch.uint8, device="cuda")
    wf.wf_skim_score(p, Q, A, W, seg, ws)
    torch.cuda.synchronize()
    for u in {0, units // 2, units - 1}:
        s = Q[0, u].double() @ A[0, u].double().T / d ** 0.5
        ref = torch.softmax(s, dim=-1).sum(0).cpu()
        check_scores(W[u], ref, f"unit {u} W")
        check_selection(seg[u].cpu(), ref, S, f"unit {u} seg")
