"""The apply step in 16 bits where a workgroup has one or two passes and its patch of W arrives before the tile of U is built: the plain form of k_decompress_wide, in blocks of 16 and of 32 rows."""
import pytest

import lsp_synth as syn
import oracle

# both sides of each line: r = 256 in blocks of 16 rows, the last column of the first pass in blocks of 32; (m, n, r, d, dtype, rows)
CASES = [
    (4101, 1024, 252, 2, "bf16", 16), (4101, 1024, 256, 2, "f16", 16), (4101, 1032, 256, 4, "bf16", 16), (4101, 8, 256, 8, "f16", 16), (4101, 1016, 512, 8, "bf16", 16), (4101, 2048, 1024, 4, "f16", 16),
    (8170, 520, 1020, 2, "bf16", 16), (16370, 1024, 260, 4, "bf16", 32), (16370, 1032, 260, 4, "f16", 32), (16370, 8, 512, 8, "bf16", 32), (16380, 1016, 288, 8, "f16", 32), (16380, 640, 512, 2, "bf16", 32),
]


def test_which_kernel_each_case_takes(tmp_path):
    from launch_routes import launches
    for (m, n, r, d, dtype, rows), calls in zip(CASES, launches([("apply", [(m, n)], r, d, dtype) for m, n, r, d, dtype, _ in CASES], str(tmp_path))):
        assert calls == [(f"k_decompress_wide<{dtype.upper()}, {rows // 16}, 4, {d}, false, 512, false, 0>", (m + rows - 1) // rows)], (m, n, r, d, dtype, calls)


@pytest.mark.gpu
@pytest.mark.parametrize("m,n,r,d,dtype,rows", CASES)
def test_apply_with_few_passes(m, n, r, d, dtype, rows):
    import gpu_util as gu
    print(f"[case] few passes m={m} n={n} r={r} d={d} {dtype}", flush=True)
    pb = syn.make_problem("few passes", m, n, r, d, dtype, seed=9700 + m + n + r + d, g_std=1.0)
    Wp, Wr = oracle.decompress_apply(pb.W, dtype, pb.S_in, pb.P_idx, pb.P_val, pb.Q_idx, pb.Q_val)
    gu.check_decompress(gu.DeviceProblem(pb).decompress(pb.S_in), pb.W, Wp, Wr, dtype, pb.name)
