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
