"""A_J of Daubechies-2 keys by the banded filter (wf_dwt_keys without details)
against the level-by-level cascade in float64."""
import math

import pytest
import torch

pytestmark = pytest.mark.gpu

R3 = math.sqrt(3.0)
G = [(1 + R3) / (4 * math.sqrt(2)), (3 + R3) / (4 * math.sqrt(2)),
     (3 - R3) / (4 * math.sqrt(2)), (1 - R3) / (4 * math.sqrt(2))]


def cascade(x, levels, boundary):
    for _ in range(levels):
        n = x.shape[1]
        ext = [n - 1, n - 2] if boundary == "symmetric" else [0, 1 % n]
        y = torch.cat([x, x[:, ext]], dim=1)
        x = sum(G[m] * y[:, m:m + n:2] for m in range(4))
    return x


# (levels, coefficients per unit): the last coefficient (J = 1) or two are edge
# ones, so one and two coefficients are all edge from J = 2 on and 3 has one
# interior one; 70 crosses a wave's run and a workgroup; past it several workgroups
# a unit.  Every block length in loads.
SHAPES = [(1, 1), (1, 2), (1, 333), (2, 1), (2, 5), (2, 300), (3, 3), (3, 70), (4, 2),
          (4, 131), (5, 4), (5, 67), (6, 1), (6, 3), (6, 35), (7, 2), (7, 19)]


@pytest.mark.parametrize("boundary", ["symmetric", "periodic"])
@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("bf16", 64), ("f32", 128), ("f32", 64)])
def test_db2_approx(dtype, d, boundary):
    import paper_2606_00724_amd as wf
    gen = torch.Generator().manual_seed(5)
    for J, n in SHAPES:
        rem = (1 << J) - 1 if n % 2 else 0  # rows past the filtered ones
        L, U = (n << J) + rem, 3
        print(f"db2 approx J={J} n={n} {dtype} d={d} {boundary}", flush=True)
        p = wf.make_params(batch=1, heads=U, ctx_len=L, head_dim=d, q_len=1, levels=J,
                           segments=1, budget=1, wavelet="db2", boundary=boundary, dtype=dtype)
        K = torch.randn((1, U, L, d), generator=gen).to(wf.torch_dtype(p))
        K[:, :, n << J:] = float("nan")  # never read
        A = wf.dwt_approx(p, K.cuda())[0].cpu().double()
        ref = cascade(K[0, :, :n << J].double(), J, boundary)
        # 3 2^J - 2 products a coefficient: batches of at most 8 rows, then
        # at most 3 2^J / 8 batches and 3 row sums, each rounded to 2^-24 of
        # partial sums below sum |f| |K|; sum |f_J| < 1.5 2^(J/2) (mirrored
        # rows at an end at most double it)
        terms = 8 + max(3, 3 * 2 ** J // 8) + 3
        bound = terms * 2.0 ** -24 * 3 * 2 ** (J / 2) * K[:, :, :n << J].abs().max().item()
        assert (A - ref).abs().max().item() <= bound


@pytest.mark.parametrize("J,d", [(1, 128), (2, 64), (2, 128), (4, 128), (6, 128)])
def test_db2_nonfinite_rows_stay_in_their_windows(J, d):
    import paper_2606_00724_amd as wf
    n, U = 41, 2
    L = n << J
    p = wf.make_params(batch=1, heads=U, ctx_len=L, head_dim=d, q_len=1, levels=J, segments=1,
                       budget=1, wavelet="db2", boundary="symmetric", dtype="bf16")
    gen = torch.Generator().manual_seed(6)
    for row in (0, (7 << J) - 1, (7 << J) - 2, (7 << J) - 3, 7 << J, L - 1):
        K = torch.randn((1, U, L, d), generator=gen).bfloat16()
        K[0, 1, row, 3] = float("nan")
        K[0, 1, row, 5] = float("inf")
        A = wf.dwt_approx(p, K.cuda())[0].cpu()
        ref = cascade(K[0].double(), J, "symmetric")
        assert torch.equal(torch.isfinite(A), torch.isfinite(ref))
