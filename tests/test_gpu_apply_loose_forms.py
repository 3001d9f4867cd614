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
    many = (4100, 1537 + 2 * d) if d >= 9 else (7200, 1665 + 2 * d) if dtype != "f32" else (4100, 1025 + 2 * d)
    return [(m, n, r, 2) for m, n, r in eight] + [(2069, 1025 + 2 * d, r, 4), (*many, r, 4)]


CASES = [(m, n, r, d, dtype, lanes) for dtype in ("bf16", "f16", "f32") for d in range(2, 13) for m, n, r, lanes in _shapes(dtype, d)
         if not (dtype != "f32" and d in (2, 4, 8, 16) and lanes == 2 and n % 2 == 0)]     # 8 rows, even rows: k_decompress
CASES += [(1037, 4098, 60, 2, "f32", 2), (1037, 4100, 67, 4, "f32", 2), (1792, 4098, 262, 8, "f32", 2), (1100, 2049, 1023, 12, "f32", 2), (13, 1037, 30, 2, "bf16", 2),
          (13, 1037, 30, 4, "f16", 2), (13, 1037, 30, 8, "bf16", 2)]


def test_which_kernel_each_case_takes(tmp_path):
    from launch_routes import launches
    for (m, n, r, d, dtype, lanes), calls in zip(CASES, launches([("apply", [(m, n)], r, d, dtype) for m, n, r, d, dtype, _ in CASES], str(tmp_path))):
        form = 1 if m > 4096 else 2
        assert len(calls) == 1 and calls[0][0] == f"k_expand_loose<{dtype.upper()}, {lanes}, {d}, false, {form}>", (m, n, r, d, dtype, calls)


# Both sides of the lines between k_expand_loose and the kernels with units of 4 rows: (m, n, r, d, dtype, whether it is the first)
LINES = [
    (4100, 3329, 30, 2, "bf16", True), (4100, 3327, 30, 3, "bf16", False), (4100, 2177, 30, 7, "f16", True), (4100, 2175, 30, 6, "bf16", False), (4100, 4097, 30, 4, "f16", False),   # 257 to 447
    (4100, 1537, 30, 9, "f16", True), (4100, 1535, 30, 9, "bf16", False), (4100, 1538, 30, 3, "bf16", True), (4100, 1534, 30, 3, "f16", False),                                      # workgroups
    (7168, 1665, 30, 4, "bf16", True), (7168, 1663, 30, 4, "f16", False), (7152, 1665, 30, 5, "bf16", False),                                                                        # and more
    (4100, 1538, 30, 4, "bf16", True), (4100, 1534, 30, 4, "f16", False), (2069, 1025, 30, 4, "f16", True), (2069, 1023, 30, 4, "bf16", False),
    (2069, 2559, 30, 4, "f32", True), (2069, 2561, 30, 4, "f32", False), (2069, 2561, 30, 5, "f32", True), (2069, 7169, 30, 8, "f32", False), (2069, 7169, 30, 7, "f32", True),
    (2069, 7168, 30, 5, "f32", True), (2069, 7170, 30, 5, "f32", False), (2069, 7170, 30, 6, "f32", True), (1040, 7167, 30, 2, "f32", True), (1040, 7169, 30, 2, "f32", False),
    (4100, 1535, 30, 4, "f32", True), (4100, 1537, 30, 4, "f32", False), (4100, 2559, 30, 5, "f32", True), (4100, 2561, 30, 5, "f32", False), (4100, 3839, 30, 8, "f32", True),
    (4100, 3841, 30, 6, "f32", False), (4100, 3841, 30, 7, "f32", True), (4100, 3841, 30, 9, "f32", True), (4100, 3840, 30, 5, "f32", True), (4100, 3842, 30, 5, "f32", False),
    (1040, 4098, 30, 4, "f32", True), (1040, 5122, 30, 4, "f32", False), (2069, 4098, 30, 4, "f32", False),
    (2069, 8192, 30, 3, "f32", True), (2069, 8208, 30, 3, "f32", False), (4100, 7200, 30, 6, "f32", True), (4100, 7184, 30, 6, "f32", False), (1040, 7200, 30, 5, "f32", True), (1040, 7184, 30, 5, "f32", False),
    (4100, 8224, 30, 9, "f32", True), (4100, 8224, 30, 4, "f32", False),                                                                                    # rows of whole lines, or not
    (2069, 511, 30, 3, "f32", True), (2069, 513, 30, 3, "f32", False), (4100, 511, 513, 3, "f32", True), (4100, 511, 512, 3, "f32", False),
]


def test_which_kernel_the_lines_give(tmp_path):
    from launch_routes import launches
    for (m, n, r, d, dtype, loose), calls in zip(LINES, launches([("apply", [(m, n)], r, d, dtype) for m, n, r, d, dtype, _ in LINES], str(tmp_path))):
        assert len(calls) == 1 and calls[0][0].startswith("k_expand_loose" if loose else "k_decompress"), (m, n, r, d, dtype, calls)
    # the bias pass has lines of its own
    bias = [(4100, 1537, 2, "bf16", True), (4100, 8191, 2, "f32", True), (4100, 4098, 2, "f32", True), (4100, 4094, 2, "f32", False)]
    for (m, n, d, dtype, loose), calls in zip(bias, launches([("bias", [(m, n)], 30, d, dtype) for m, n, d, dtype, _ in bias], str(tmp_path))):
        assert calls[0][0].startswith("k_expand_loose" if loose else "k_decompress"), (m, n, d, dtype, calls)


@pytest.mark.gpu
@pytest.mark.parametrize("m,n,r,d,dtype,loose", LINES)
def test_apply_on_both_sides_of_the_lines(m, n, r, d, dtype, loose):
    test_apply_in_every_form(m, n, r, d, dtype, None)


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
