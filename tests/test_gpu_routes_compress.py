"""Kernel B of compress in two rounds over the columns (slices of T beyond 4 MB; r = 1024, 1536 and 2048, and others above 1536 up to 9 MB with d >= 4), alone and in groups with matrices of one round; which shapes take how many."""
import pytest

import lsp_synth as syn


def _grid(m, r, d, rounds):
    items = r + (m * d + 255) // 256 + 1                              # the most pieces that the rows of P^T can be cut into
    return 8 * rounds * ((items + 3) // 4)


# (shapes, r, d, dtype, the launches of kernel B: lanes a group, workgroups)
ROUTES = [
    ([(8200, 40)], 2048, 3, "f16", [(32, _grid(8200, 2048, 3, 2))]),
    ([(8200, 40)], 2047, 3, "f16", [(64, _grid(8200, 2047, 3, 1))]),          # no whole lines of 128 bytes
    ([(8200, 40)], 2047, 4, "f16", [(32, _grid(8200, 2047, 4, 2))]),          # ... but lists long enough
    ([(9221, 40)], 2047, 4, "f16", [(64, _grid(9221, 2047, 4, 1))]),          # ... and too much
    ([(6000, 40)], 1540, 8, "bf16", [(32, _grid(6000, 1540, 8, 2))]), ([(6000, 40)], 1532, 8, "bf16", [(64, _grid(6000, 1532, 8, 1))]),
    ([(4097, 24)], 2048, 2, "bf16", [(32, _grid(4097, 2048, 2, 2))]),
    ([(4096, 24)], 2048, 2, "bf16", [(64, _grid(4096, 2048, 2, 1))]),
    ([(5462, 24)], 1536, 2, "f32", [(32, _grid(5462, 1536, 2, 2))]),
    ([(5461, 24)], 1536, 2, "f32", [(64, _grid(5461, 1536, 2, 1))]),
    ([(8193, 16)], 1024, 2, "f32", [(16, _grid(8193, 1024, 2, 2))]),
    ([(8192, 16)], 1024, 2, "f32", [(32, _grid(8192, 1024, 2, 1))]),
    ([(16400, 16)], 1030, 2, "f32", [(64, _grid(16400, 1030, 2, 1))]),
    ([(17000, 8)], 512, 4, "f32", [(16, _grid(17000, 512, 4, 1))]),           # stripes of 32 columns would leave half of the lanes idle
    ([(700, 41), (8200, 40)], 2048, 3, "f16", [(64, _grid(700, 2048, 3, 1)), (32, _grid(8200, 2048, 3, 2))]),
    ([(8200, 24), (4104, 40), (700, 41), (8300, 16)], 2048, 2, "f32",
     [(64, _grid(700, 2048, 2, 1)), (32, _grid(4104, 2048, 2, 2) + _grid(8200, 2048, 2, 2) + _grid(8300, 2048, 2, 2))]),
]


def test_rounds_of_every_shape(tmp_path):
    from launch_routes import launches
    found = launches([("compress", shapes, r, d, dtype) for shapes, r, d, dtype, _ in ROUTES], str(tmp_path))
    for (shapes, r, d, dtype, want), calls in zip(ROUTES, found):
        assert [x for x in calls if "pt8" in x[0]] == [(f"k_compress_pt8<{lanes}>", grid) for lanes, grid in want], (shapes, r, d, dtype, calls)


@pytest.mark.gpu
@pytest.mark.parametrize("m,n,r,d,dtype", [(8200, 40, 2048, 3, "f16"), (4097, 24, 2048, 2, "bf16"), (5462, 24, 1536, 3, "f32"), (8193, 24, 1024, 2, "bf16"), (16400, 24, 1024, 1, "f16"),
                                            (8200, 24, 2047, 4, "f16"), (6000, 24, 1540, 5, "bf16")])
def test_compress_in_two_rounds(m, n, r, d, dtype):
    from test_gpu_rounds import test_compress_in_rounds
    test_compress_in_rounds(m, n, r, d, dtype, "uniform")             # alone against the oracle, and bit for bit in a group with a matrix of one round


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["bf16", "f16", "f32"])
def test_a_group_of_one_round_and_two(dtype):
    import torch
    import gpu_util as gu
    import oracle
    import paper_2406_10181_amd as lsp
    shapes, r, d = ROUTES[-1][:3]
    print(f"[case] one and two rounds {dtype}", flush=True)
    dps = [gu.DeviceProblem(syn.make_problem("rounds", m, n, r, d, dtype, seed=9920 + m, g_std=1.0)) for m, n in shapes]
    singles = [dp.compress_planned() for dp in dps]
    for dp, S in zip(dps, singles):
        pb = dp.pb
        gu.check_compress(S, oracle.compress(pb.G, pb.dtype, pb.P_idx, pb.P_val, pb.Q_idx, pb.Q_val, pb.r), "alone")
        dp.S.fill_(float("nan"))
    items = [(x.G, x.plan, x.S, x.ws, x.ws_bytes, x.pb.m, x.pb.n) for x in dps]
    lsp.lsp_compress_planned_grouped(lsp.compress_items(items), len(items), r, d, dps[0].code, torch.cuda.current_stream())
    torch.cuda.synchronize()
    for dp, S in zip(dps, singles):
        assert (dp.S.cpu().numpy() == S).all()
