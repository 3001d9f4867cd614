"""Kernel B of compress where its slices of T are larger than an XCD's L2, in one round over the columns or two, with a last stripe that is not whole, beside a matrix of one round in a group; and its groups of eight lanes."""
import pytest

import lsp_synth as syn
import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,n,r,d,dtype,dist", [
    (4104, 24, 2048, 2, "bf16", "uniform"),      # just over 4 MB a slice: two rounds of 32 quads
    (8200, 40, 2047, 3, "f16", "uniform"),       # one round of 64, its last stripe not whole (r is no multiple of 512, and d < 4)
    (16400, 16, 1030, 2, "f32", "uniform"),      # one round of 33 quads, 27 in the last stripe
    (20000, 8, 520, 4, "f32", "uniform"),        # stripes of 64 columns at the least: one round
    (9000, 40, 1100, 4, "f32", "zipf"),          # rows of P^T cut into pieces
])
def test_compress_in_rounds(m, n, r, d, dtype, dist):
    import gpu_util as gu
    print(f"[case] rounds m={m} n={n} r={r} d={d} {dtype}", flush=True)
    pb = syn.make_problem("rounds", m, n, r, d, dtype, seed=9900 + r, g_std=1.0, index_dist=dist)
    dp = gu.DeviceProblem(pb)
    S_o = oracle.compress(pb.G, pb.dtype, pb.P_idx, pb.P_val, pb.Q_idx, pb.Q_val, pb.r)
    S = dp.compress_planned()
    gu.check_compress(S, S_o, "rounds")
    if dist == "uniform":                         # (nothing added with atomics)
        import torch
        import paper_2406_10181_amd as lsp
        small = gu.DeviceProblem(syn.make_problem("one round", 700, n + 1, r, d, dtype, seed=3, g_std=1.0))
        small.build_plan()
        items = [(x.G, x.plan, x.S, x.ws, x.ws_bytes, x.pb.m, x.pb.n) for x in (small, dp)]
        lsp.lsp_compress_planned_grouped(lsp.compress_items(items), 2, r, d, dp.code, torch.cuda.current_stream())
        torch.cuda.synchronize()
        assert (dp.S.cpu().numpy() == S).all()
        together = small.S.cpu().numpy()
        assert (small.compress_planned() == together).all()


@pytest.mark.parametrize("m,n,r,d,dtype,dist", [
    (40, 24, 4, 1, "f32", "uniform"),            # one stripe has a column; rows of some ten entries
    (520, 40, 16, 8, "bf16", "uniform"),         # pieces of 256 entries: whole batches of 64, and a last one
    (700, 24, 33, 3, "f16", "zipf"),             # the last quad overlaps the one before
    (130, 24, 255, 2, "f32", "uniform"),         # eight lanes, the last quad short; rows without an entry
    (64, 300, 256, 64, "bf16", "uniform"),
    (130, 24, 257, 4, "f32", "uniform"),         # nine quads a stripe: sixteen lanes
])
def test_compress_with_eight_lanes_a_row(m, n, r, d, dtype, dist):
    import gpu_util as gu
    print(f"[case] eight lanes m={m} n={n} r={r} d={d} {dtype} {dist}", flush=True)
    pb = syn.make_problem("eight", m, n, r, d, dtype, seed=9950 + r, g_std=1.0, index_dist=dist)
    dp = gu.DeviceProblem(pb)
    gu.check_compress(dp.compress_planned(), oracle.compress(pb.G, pb.dtype, pb.P_idx, pb.P_val, pb.Q_idx, pb.Q_val, pb.r), "eight")
