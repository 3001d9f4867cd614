"""The tile U = P S of the apply step where its work items (a row of the tile, four columns) are one, just over one and several for a thread, taken
singly or together, against the oracle."""
import pytest

import lsp_synth as syn
import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f16", "f32"])
@pytest.mark.parametrize("d", [2, 4, 8])
@pytest.mark.parametrize("m,r", [
    (13, 9), (13, 255), (13, 256), (13, 257), (13, 514), (13, 1021),     # 4 rows
    (2069, 9), (2069, 128), (2069, 130), (2069, 384), (2069, 511),      # 16 rows: up to 128 columns
    (13, 1025), (13, 1100), (13, 1400), (13, 2047), (13, 2048), (2069, 1536),   # row by row, or in stripes of 256 columns
])
def test_apply_with_few_and_many_items_a_thread(m, r, d, dtype):
    import gpu_util as gu
    pb = syn.make_problem("tile", m, 66, r, d, dtype, seed=9000 + m + r + d, g_std=1.0)
    print(f"[case] tile m={m} r={r} d={d} {dtype}", flush=True)
    Wp, Wr = oracle.decompress_apply(pb.W, dtype, pb.S_in, pb.P_idx, pb.P_val, pb.Q_idx, pb.Q_val)
    gu.check_decompress(gu.DeviceProblem(pb).decompress(pb.S_in), pb.W, Wp, Wr, dtype, pb.name)


# What the kernel for whole pieces of 8 columns does at its edges: one piece, a pass and a bit, less than a block of rows more; blocks of 4 rows (m = 13, d <= 8, r <= 1024;
# k_decompress) or 8 (m = 13, other d and r), of 16 on one workgroup a CU (2069) and on more (4100), of 32 (16390).  Against the oracle, and bit for bit what the other kernel makes of the same matrix: a group with a ragged matrix goes there.
@pytest.mark.parametrize("dtype", ["bf16", "f16", "f32"])
@pytest.mark.parametrize("d", [2, 4, 8, 16])
@pytest.mark.parametrize("m,n,r", [(13, 8, 16), (13, 1032, 132), (13, 520, 1540), (2069, 8, 20), (2069, 520, 260), (2069, 1544, 1024), (4100, 72, 512), (16390, 24, 260), (16390, 520, 512)])
def test_apply_in_whole_pieces(m, n, r, d, dtype):
    import torch
    import gpu_util as gu
    import paper_2406_10181_amd as lsp
    print(f"[case] pieces m={m} n={n} r={r} d={d} {dtype}", flush=True)
    pb = syn.make_problem("pieces", m, n, r, d, dtype, seed=9500 + m + n + r + d, g_std=1.0)
    Wp, Wr = oracle.decompress_apply(pb.W, dtype, pb.S_in, pb.P_idx, pb.P_val, pb.Q_idx, pb.Q_val)
    dp = gu.DeviceProblem(pb)
    single = dp.decompress(pb.S_in)
    gu.check_decompress(single, pb.W, Wp, Wr, dtype, pb.name)
    other = gu.DeviceProblem(syn.make_problem("ragged", 33, 66, r, d, dtype, seed=1, g_std=1.0))
    S = gu.to_device(pb.S_in)
    items = [(x.W, S, x.P_idx, x.P_val, x.Q_idx, x.Q_val, x.pb.m, x.pb.n) for x in (dp, other)]
    lsp.lsp_decompress_apply_grouped(lsp.apply_items(items), 2, r, d, dp.code, torch.cuda.current_stream())
    torch.cuda.synchronize()
    assert (gu.to_host(dp.W, dtype) == single).all()


# d = 16 in blocks of 8 rows on more workgroups than CUs (r > 1024 only), against the oracle.
@pytest.mark.parametrize("dtype", ["bf16", "f16", "f32"])
@pytest.mark.parametrize("m,n,r", [(2100, 520, 1540), (2053, 1032, 2048)])
def test_apply_and_bias_with_a_large_tile_of_8_rows(m, n, r, dtype):
    import gpu_util as gu
    from test_gpu_parity import _bias_check
    print(f"[case] large tile m={m} n={n} r={r} {dtype}", flush=True)
    pb = syn.make_problem("large tile", m, n, r, 16, dtype, seed=9700 + m + n + r, g_std=1.0)
    Wp, Wr = oracle.decompress_apply(pb.W, dtype, pb.S_in, pb.P_idx, pb.P_val, pb.Q_idx, pb.Q_val)
    gu.check_decompress(gu.DeviceProblem(pb).decompress(pb.S_in), pb.W, Wp, Wr, dtype, pb.name)
    _bias_check(pb)


# The bias pass in the same kernel: one piece, part passes, last blocks that are not whole (a lane past the last column still has sums, which must not
# count), on one workgroup a CU (2069) and on more (4100, 8200).
@pytest.mark.parametrize("dtype", ["bf16", "f16", "f32"])
@pytest.mark.parametrize("d", [2, 4, 8, 16])
@pytest.mark.parametrize("m,n,r", [(13, 8, 16), (13, 1032, 132), (2069, 8, 20), (2069, 520, 260), (2069, 1544, 1024), (4100, 72, 512), (4100, 1544, 256), (8200, 264, 1024)])
def test_bias_in_whole_pieces(m, n, r, d, dtype):
    from test_gpu_parity import _bias_check
    _bias_check(syn.make_problem("bias pieces", m, n, r, d, dtype, seed=9600 + m + n + r + d, g_std=1.0))


# Passes that take turns with two sets of registers: one to four of them, on one workgroup a CU (2069), on one or two (4100) and on workgroups of 256 threads (8200).
@pytest.mark.parametrize("dtype", ["bf16", "f16", "f32"])
@pytest.mark.parametrize("d", [2, 4, 8])
@pytest.mark.parametrize("m,n,r", [(2069, 3080, 260), (4100, 2056, 260), (4100, 3072, 132), (8200, 264, 132), (8200, 1032, 132), (8200, 2048, 260)])
def test_apply_and_bias_over_several_passes(m, n, r, d, dtype):
    from test_gpu_parity import _bias_check
    test_apply_in_whole_pieces(m, n, r, d, dtype)
    _bias_check(syn.make_problem("bias passes", m, n, r, d, dtype, seed=9800 + m + n + r + d, g_std=1.0))


# Both sides of the rules for the rows of a workgroup where k_decompress_wide serves: 129 to 255 blocks of 16 rows, and 1024 and more.
@pytest.mark.parametrize("m,n,r,d,dtype", [
    (2069, 1024, 128, 2, "f32"), (2069, 1032, 260, 4, "f32"), (2069, 1032, 128, 2, "f32"), (2069, 1024, 132, 2, "f32"),
    (2069, 8192, 256, 2, "bf16"), (2069, 8192, 260, 2, "f16"), (2069, 8184, 256, 2, "bf16"), (2069, 8192, 256, 4, "bf16"),
    (16390, 2040, 260, 2, "bf16"), (16390, 2048, 260, 2, "f16"), (16390, 2048, 260, 4, "bf16"), (16390, 2048, 260, 8, "f16"),
])
def test_apply_and_bias_on_both_sides_of_the_rules_for_whole_pieces(m, n, r, d, dtype):
    from test_gpu_parity import _bias_check
    test_apply_in_whole_pieces(m, n, r, d, dtype)
    _bias_check(syn.make_problem("bias rules", m, n, r, d, dtype, seed=9900 + m + n + r + d, g_std=1.0))
