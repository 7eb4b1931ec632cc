"""Which parameters the fused calls take does not depend on how a plan splits
the work (no GPU needed: plans are host arithmetic over 256 CUs)."""
import pytest


@pytest.mark.parametrize("units,J,L,B,S,k,taken", [
    (76, 6, 14832, 256, 118, 4587, True),    # 3 ranges of 4096 positions would not fit the LDS
    (210, 8, 3196, 256, 10, 928, True),
    (83, 5, 24967, 256, 266, 3564, True),
    (76, 6, 14832, 64, 118, 4587, True),
    (373, 8, 10252, 256, 18, 1318, False),   # one range of 4096 positions: never fitted
    (389, 6, 46747, 256, 75, 2974, False),
])
def test_large_query_blocks(units, J, L, B, S, k, taken):
    import paper_2606_00724_amd as wf
    p = wf.make_params(batch=1, heads=units, ctx_len=L, head_dim=128, q_len=B, levels=J,
                       segments=S, budget=k, dtype="bf16")
    for op in (wf.OP_FUSED, wf.OP_CACHED, wf.OP_SHARED):
        assert (wf.workspace_bytes(p, op) > 0) == taken
