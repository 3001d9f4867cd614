"""k_expand_loose in every form that the apply step has (blocks of 8 rows, of 16 on one workgroup a CU and on more) and for every d from 2 to 12; in fp32 blocks of 8 rows serve 65 to 128
blocks of 16."""
import pytest

import lsp_synth as syn
import oracle

# (dtype, d) -> shapes of the three forms: n odd or even, r with a last quad of every length
def _shapes(dtype, d):
    r = 21 + 47 * d % 64
    eight = [(1037, 1024 + d | 1, r)] if dtype == "f32" else [(13, 1024 + d, r)]
    if dtype == "f32" and d % 2:
        eight.append((1100, 490 + d, r + 1))
    return [(m, n, r, 2) for m, n, r in eight] + [(2069, 1025 + 2 * d, r, 4), (4100, 1537 + 2 * d, r, 4)]


CASES = [(m, n, r, d, dtype, lanes) for dtype in ("bf16", "f16", "f32") for d in range(2, 13) for m, n, r, lanes in _shapes(dtype, d)
         if not (dtype != "f32" and d in (2, 4, 8, 16) and lanes == 2 and n % 2 == 0)]     # 8 rows, even rows: k_decompress
CASES += [(1037, 4098, 60, 2, "f32", 2), (1037, 4100, 67, 4, "f32", 2), (1792, 4098, 262, 8, "f32", 2), (1100, 2049, 1023, 12, "f32", 2), (13, 1037, 30, 2, "bf16", 2),
          (13, 1037, 30, 4, "f16", 2), (13, 1037, 30, 8, "bf16", 2)]


def test_which_kernel_each_case_takes(tmp_path):
    from launch_routes import launches
    for (m, n, r, d, dtype, lanes), calls in zip(CASES, launches([("apply", [(m, n)], r, d, dtype) for m, n, r, d, dtype, _ in CASES], str(tmp_path))):
        form = 1 if m > 4096 else 2
        assert len(calls) == 1 and calls[0][0] == f"k_expand_loose<{dtype.upper()}, {lanes}, {d}, false, {form}>", (m, n, r, d, dtype, calls)


@pytest.mark.gpu
@pytest.mark.parametrize("m,n,r,d,dtype,lanes", CASES)
def test_apply_in_every_form(m, n, r, d, dtype, lanes):
    import gpu_util as gu
    print(f"[case] loose form m={m} n={n} r={r} d={d} {dtype}", flush=True)
    pb = syn.make_problem("loose form", m, n, r, d, dtype, seed=9300 + m + n + r + d, g_std=1.0)
    Wp, Wr = oracle.decompress_apply(pb.W, dtype, pb.S_in, pb.P_idx, pb.P_val, pb.Q_idx, pb.Q_val)
    gu.check_decompress(gu.DeviceProblem(pb).decompress(pb.S_in), pb.W, Wp, Wr, dtype, pb.name)


@pytest.mark.gpu
@pytest.mark.parametrize("m,n,r,d", [(1037, 1031, 23, 7), (1100, 4098, 262, 8), (1793, 1029, 21, 3), (1040, 301, 50, 9)])
def test_nothing_beside_the_matrix_is_touched_in_blocks_of_8_rows(m, n, r, d):
    from test_gpu_apply_loose import test_nothing_beside_the_matrix_is_touched
    test_nothing_beside_the_matrix_is_touched(m, n, r, d, "f32")
