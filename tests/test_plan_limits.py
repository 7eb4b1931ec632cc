"""Which parameters the fused calls take does not depend on how a plan splits
the work, and which splits are taken (no GPU needed: plans are host arithmetic
over 256 CUs)."""
import os
import subprocess

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


def _ranges(wf, units, rows, B):
    """fp32 ranges of a unit's pool of `rows` positions (64 channels), from the
    statistics that the staged scan asks for beside the weights"""
    p = wf.make_params(batch=1, heads=units, ctx_len=8192, head_dim=64, q_len=B, levels=3,
                       segments=rows // 8, budget=rows, dtype="f32")

    def up(x):
        return (x + 255) & ~255
    need = wf.workspace_bytes(p, wf.OP_SCAN) - up(units * rows * 4)
    for c in range(1, 1025):
        if up(units * c * 2 * B * 4) == need:
            return c
    raise AssertionError(need)


@pytest.mark.parametrize("units,rows", [(129, 1000), (171, 4000), (265, 512), (265, 1000),
                                        (300, 4000), (129, 4000)])
def test_fp32_rounds_leave_few_cus_idle(units, rows):
    """A round of workgroups lasts as long as its longest: rounds times a
    workgroup's chunks (and one for its constant part).  Where one range a unit
    would leave much of its last round idle, the chosen count costs at least
    15% less."""
    import paper_2606_00724_amd as wf
    chunks = (rows + 63) // 64

    def cost(c):
        per = -(-chunks // c)
        return -(-units * -(-chunks // per) // 256) * (per + 1)
    assert cost(_ranges(wf, units, rows, 64)) <= 0.85 * cost(1)


@pytest.mark.parametrize("dtype,B,L,apart", [
    ("bf16", 16, 7933 * 16, True),    # coefficients no multiple of four
    ("bf16", 100, 8192 * 16, True), ("f32", 16, 8192 * 16, True),
    ("bf16", 16, 8192 * 16, False),
    ("f32", 16, 1024 * 16, False), ("bf16", 100, 1024 * 16, False)])
def test_large_pools_are_selected_apart(dtype, B, L, apart):
    """Pools past 16384 positions are not selected by every workgroup of the
    attention where a kernel of its own used to do it."""
    import paper_2606_00724_amd as wf
    S = (L >> 4) * 7 // 8
    p = wf.make_params(batch=1, heads=5, ctx_len=L, head_dim=128, q_len=B, levels=4, segments=S,
                       budget=4 * S, dtype=dtype, wavelet="db2")
    assert ("scan_select" in wf.fused_kernel_names(p)) == apart


# (kernel, units, chunks, workgroups resident at once, most chunks a range) of
# the longer-range cases of test_gpu_dispatch_edges.py: 16384 keys and 11520 pool
# positions in chunks of 128, 5760 rows in chunks of 64; fp32: 2560 in chunks of 64
LONGER = [("token skim", 28, 128, 512, 128), ("held and db2 skims", 28, 128, 256, 128),
          ("bf16 scan", 28, 90, 256, 32), ("bf16 attention", 28, 90, 256, 64),
          ("fp32 scan", 40, 40, 256, 0), ("fp32 attention", 40, 40, 256, 0)]


def test_odd_unit_counts_take_fewer_longer_ranges(tmp_path):
    """Each kernel's plan takes less than ceil(resident / units) ranges a unit, and
    ranges of more chunks than that count would give."""
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    src = tmp_path / "ranges.cpp"
    body = "".join(
        f'  std::printf("%ld\\n", ' + (
            f"wf::ranges_per_unit({u}, {c}, {slots}, {most})" if most else
            f"wf::fp32_ranges_per_unit({u}, {c}, {slots}, {c}, 1)") + ");\n"
        for _, u, c, slots, most in LONGER)
    src.write_text('#include <cstdio>\nnamespace wf { struct Db2TokenTaps; }\n#include "wf_launch.hpp"\n'
                   "namespace wf { int device_cu_count() { return 256; } }\n"
                   "int main() {\n" + body + "}\n")
    exe = tmp_path / "ranges"
    subprocess.run(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    f"-I{root}/include", f"-I{root}/paper_2606_00724_amd/csrc", str(src), "-o",
                    str(exe)], check=True)
    got = [int(x) for x in subprocess.run([str(exe)], capture_output=True, text=True,
                                          check=True).stdout.split()]
    for (name, units, chunks, slots, _), ranges in zip(LONGER, got):
        up = -(-slots // units)
        assert ranges < up, name
        assert -(-chunks // ranges) > -(-chunks // up), name
