"""The apply step in blocks of 8 rows, which 65 to 128 blocks of 16 rows take (fewer take blocks of 4): the edges of the tile of U in k_decompress and k_decompress_any."""
import pytest

import lsp_synth as syn
import oracle

# up to 256 columns there is one item of the tile a thread; r in planes of 256, 512 and 1024 columns
TILES = [(m, 66, r, d, dtype) for dtype in ("f16", "f32") for d in (2, 4, 8) for m, r in ((1037, 9), (1037, 255), (1037, 256), (1037, 257), (1037, 514), (1037, 1021))]
WHOLE = [(m, n, r, d, dtype) for dtype in ("bf16", "f16", "f32") for d in (2, 4, 8) for m, n, r in ((1037, 8, 16), (1037, 1032, 132), (1789, 520, 600))]
ANY = [(1037, 67, 300, 5, "f16"), (1037, 66, 21, 3, "bf16"), (1050, 261, 900, 5, "bf16"), (1050, 1024, 31, 13, "f32"), (1100, 67, 600, 64, "f32"), (1037, 1030, 250, 17, "f16")]


def test_which_kernel_each_case_takes(tmp_path):
    from launch_routes import launches
    cases = TILES + WHOLE + ANY
    for case, calls in zip(cases, launches([("apply", [(m, n)], r, d, dtype) for m, n, r, d, dtype in cases], str(tmp_path))):
        m, n, r, d, dtype = case
        plane = 4096 if r <= 256 else 8192 if r <= 512 else 16384
        kernel = f"k_decompress_any<{dtype.upper()}, 2, {plane}, 512, {'true' if n % 2 == 0 else 'false'}, false>" if case in ANY else f"k_decompress<{dtype.upper()}, 2, {d}, {plane}, 512, false>"
        assert calls == [(kernel, (m + 7) // 8)], (case, calls)
    few = [(13, 66, 257, 4, "f16"), (1024, 66, 257, 4, "f32"), (1793, 66, 257, 4, "f32")]         # these have blocks of 4 rows
    for case, calls in zip(few, launches([("apply", [(m, n)], r, d, dtype) for m, n, r, d, dtype in few], str(tmp_path))):
        assert calls == [(f"k_decompress<{case[4].upper()}, 1, 4, 8192, 512, false>", (case[0] + 3) // 4)], (case, calls)


@pytest.mark.gpu
@pytest.mark.parametrize("m,n,r,d,dtype", TILES + WHOLE + ANY)
def test_apply_in_blocks_of_8_rows(m, n, r, d, dtype):
    import gpu_util as gu
    print(f"[case] 8 rows m={m} n={n} r={r} d={d} {dtype}", flush=True)
    pb = syn.make_problem("8 rows", m, n, r, d, dtype, seed=9200 + m + n + r + d, g_std=1.0)
    Wp, Wr = oracle.decompress_apply(pb.W, dtype, pb.S_in, pb.P_idx, pb.P_val, pb.Q_idx, pb.Q_val)
    gu.check_decompress(gu.DeviceProblem(pb).decompress(pb.S_in), pb.W, Wp, Wr, dtype, pb.name)


# Blocks of 4 rows or of 8: at most 64 blocks of 16 with lists of more than 12 entries, whose passes are shared, and fp32 with 113 to 128 blocks: (m, n, r, d, dtype, rows, workgroups a block)
FOUR_OR_EIGHT = [
    (1000, 513, 60, 13, "bf16", 8, 1), (1000, 512, 60, 13, "f32", 4, 1), (1000, 2049, 60, 20, "f16", 8, 2), (100, 5003, 70, 64, "f32", 8, 5), (100, 5003, 70, 12, "f32", 4, 5), (37, 4099, 300, 17, "bf16", 8, 5),
    (5, 6001, 600, 33, "bf16", 8, 6), (513, 3075, 900, 14, "f32", 8, 2),
    (2048, 6144, 260, 4, "f32", 4, 1), (2048, 6146, 260, 4, "f32", 8, 1), (2048, 4096, 260, 8, "f32", 4, 1), (2048, 5122, 258, 8, "f32", 8, 1), (1793, 4094, 60, 8, "f32", 8, 1),
]


def test_which_kernel_has_blocks_of_4_rows_and_of_8(tmp_path):
    from launch_routes import launches
    for (m, n, r, d, dtype, rows, parts), calls in zip(FOUR_OR_EIGHT, launches([("apply", [(m, n)], r, d, dtype) for m, n, r, d, dtype, _, _ in FOUR_OR_EIGHT], str(tmp_path))):
        kernel = f"k_decompress_any<{dtype.upper()}, {rows // 4}, " if d > 8 else f"k_decompress<{dtype.upper()}, {rows // 4}, {d}, "
        assert len(calls) == 1 and calls[0][0].startswith(kernel) and calls[0][1] == (m + rows - 1) // rows * parts, (m, n, r, d, dtype, calls)


@pytest.mark.gpu
@pytest.mark.parametrize("m,n,r,d,dtype,rows,parts", FOUR_OR_EIGHT)
def test_apply_in_blocks_of_4_rows_and_of_8(m, n, r, d, dtype, rows, parts):
    test_apply_in_blocks_of_8_rows(m, n, r, d, dtype)
