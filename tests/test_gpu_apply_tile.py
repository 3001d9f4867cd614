"""The tile U = P S of the apply step where its work items (a row of the tile, four columns) are one, just over one and several for a thread, taken
singly or together, against the oracle."""
import pytest

import lsp_synth as syn
import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f16", "f32"])
@pytest.mark.parametrize("d", [2, 4, 8])
@pytest.mark.parametrize("m,r", [
    (13, 9), (13, 255), (13, 256), (13, 257), (13, 514), (13, 1021),     # 8 rows: up to 256 columns there is one item a thread
    (2069, 9), (2069, 128), (2069, 130), (2069, 384), (2069, 511),      # 16 rows: up to 128 columns
    (13, 1025), (13, 1100), (13, 1400), (13, 2047), (13, 2048), (2069, 1536),   # row by row, or in stripes of 256 columns
])
def test_apply_with_few_and_many_items_a_thread(m, r, d, dtype):
    import gpu_util as gu
    pb = syn.make_problem("tile", m, 66, r, d, dtype, seed=9000 + m + r + d, g_std=1.0)
    print(f"[case] tile m={m} r={r} d={d} {dtype}", flush=True)
    Wp, Wr = oracle.decompress_apply(pb.W, dtype, pb.S_in, pb.P_idx, pb.P_val, pb.Q_idx, pb.Q_val)
    gu.check_decompress(gu.DeviceProblem(pb).decompress(pb.S_in), pb.W, Wp, Wr, dtype, pb.name)
