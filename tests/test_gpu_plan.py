"""The device-side plan build against the host builder: the same bytes, for every shape class the plan has
(one slot with dealt lists, several slots, shared columns, spare lanes, cut rows of P^T, ragged chunks), and
its error reporting."""
import numpy as np
import pytest

import lsp_synth as syn

pytestmark = pytest.mark.gpu


def _both(m, n, r, d, dist, seed):
    import torch
    import paper_2406_10181_amd as L
    rng = np.random.default_rng(seed)
    P_idx, P_val = syn.ell_projector(m, r, d, rng, dist)
    Q_idx, Q_val = syn.ell_projector(n, r, d, rng, dist)
    nb = L.lsp_plan_bytes(m, n, r, d)
    host = np.zeros(nb, dtype=np.uint8)
    rc_host = L.lsp_plan_build_host(P_idx, P_val, Q_idx, Q_val, m, n, r, d, host, nb, check=False)
    dev = [torch.from_numpy(x).cuda() for x in (P_idx, P_val, Q_idx, Q_val)]
    plan = torch.full((nb,), 0xA5, dtype=torch.uint8, device="cuda")
    wb = L.lsp_plan_build_workspace_bytes(m, n, r, d)
    ws = torch.empty(wb, dtype=torch.uint8, device="cuda")
    status = torch.full((1,), 77, dtype=torch.int32, device="cuda")
    L.lsp_plan_build_async(*dev, m, n, r, d, plan, nb, ws, wb, status, torch.cuda.current_stream())
    torch.cuda.synchronize()
    return rc_host, host, int(status.item()), plan.cpu().numpy(), dev


@pytest.mark.parametrize("m,n,r,d,dist", [
    (48, 4200, 16, 2, "distinct"),      # three chunks, ragged last chunk, spare lanes handed out
    (40, 2048, 64, 4, "uniform"),
    (33, 2500, 96, 8, "zipf"),          # hot columns get several owners; long rows of P^T are cut
    (2000, 64, 4, 2, "uniform"),        # every row of P^T has ~1000 entries -> pieces + atomic flag
    (24, 3000, 600, 2, "uniform"),      # more columns than lanes: two slots
    (10, 7, 3, 1, "uniform"),
    (1, 1, 1, 1, "uniform"),
    (300, 6152, 256, 4, "uniform"),     # spare lanes: half the columns get a second owner
    (2048, 2048, 1280, 4, "uniform"),   # three slots
    (4096, 4096, 512, 8, "uniform"),    # a square matrix of the 6.7B-style stack
    (4096, 11008, 512, 8, "uniform"),   # its wide matrix
    (11008, 4096, 512, 8, "uniform"),   # its tall matrix
    (4096, 16384, 256, 16, "zipf"),     # wide sweep, most skewed point
    (4096, 16384, 1024, 2, "zipf"),
    (4096, 4096, 2048, 8, "uniform"),   # four slots
])
def test_device_plan_equals_host_plan(m, n, r, d, dist):
    print(f"[case] device plan m={m} n={n} r={r} d={d} {dist}", flush=True)
    rc_host, host, rc_dev, dev_plan, _ = _both(m, n, r, d, dist, seed=8800 + m + n + r)
    assert rc_host == 0 and rc_dev == 0
    bad = np.flatnonzero(host != dev_plan)
    assert bad.size == 0, f"{bad.size} bytes differ, first at offset {bad[:4]}"


@pytest.mark.parametrize("m,n,r,d,dist", [
    (2049, 2047, 33, 1, "uniform"),     # a tile of one row; a part of the sort smaller than one wave's step
    (257, 2304, 1, 1, "uniform"),       # one column: every entry of a step of 64 meets every other
    (300, 2303, 2048, 64, "uniform"),   # the most columns and the most entries a tile can have
    (4097, 513, 512, 3, "zipf"),        # three tiles of P, parts that end inside a step
    (9, 4100, 64, 64, "distinct"),      # by length: 512 lists of 256 entries, and of one or none in the last chunk
    (9, 4200, 600, 64, "uniform"),      # two slots, lists on both sides of 256 entries
    (9, 2200, 1000, 40, "zipf"),        # three or four slots of lists of all lengths
    (9, 2100, 1500, 2, "zipf"),         # mostly empty lists
])
def test_device_plan_at_the_edges_of_the_sort(m, n, r, d, dist):
    print(f"[case] device plan m={m} n={n} r={r} d={d} {dist}", flush=True)
    rc_host, host, rc_dev, dev_plan, _ = _both(m, n, r, d, dist, seed=77 + m + n + r)
    assert rc_host == rc_dev
    if rc_host == 0:
        bad = np.flatnonzero(host != dev_plan)
        assert bad.size == 0, f"{bad.size} bytes differ, first at offset {bad[:4]}"


def test_device_plan_and_new_values_with_values_of_every_magnitude():
    """The parts of a value on the device (build and refresh) against the host's: subnormal, large, infinite and no numbers."""
    import torch
    import paper_2406_10181_amd as L
    m, n, r, d = 40, 2500, 96, 8
    rng = np.random.default_rng(8899)
    P_idx, P_val = syn.ell_projector(m, r, d, rng)
    Q_idx, Q_val = syn.ell_projector(n, r, d, rng)
    wide = (np.ldexp(rng.uniform(1.0, 2.0, (n, d)), rng.integers(-150, 128, (n, d))) * rng.choice([-1.0, 1.0], (n, d))).astype(np.float32)
    wide.reshape(-1)[:8] = np.array([0, 0x80000000, 1, 0x7F7FFFFF, 0x7F800000, 0xFF800000, 0x7F800001, 0xFFC12345], np.uint32).view(np.float32)
    print("[case] device plan, values of every magnitude", flush=True)
    nb = L.lsp_plan_bytes(m, n, r, d)
    host = np.zeros(nb, dtype=np.uint8)
    assert L.lsp_plan_build_host(P_idx, P_val, Q_idx, wide, m, n, r, d, host, nb, check=False) == 0
    P_idx, P_val, Q_idx, Q_val, wide = [torch.from_numpy(x).cuda() for x in (P_idx, P_val, Q_idx, Q_val, wide)]
    stream = torch.cuda.current_stream()
    for values in (wide, Q_val):
        plan = torch.empty(nb, dtype=torch.uint8, device="cuda")
        L.lsp_plan_build(P_idx, P_val, Q_idx, values, m, n, r, d, plan, nb, stream)
        if values is Q_val:
            L.lsp_plan_refresh_values(plan, P_val, wide, m, n, r, d, stream)
        torch.cuda.synchronize()
        assert np.array_equal(plan.cpu().numpy(), host)


def test_device_plan_reports_skew_and_bad_indices():
    import torch
    import paper_2406_10181_amd as L
    # r = 2048 uniformly used columns fill all 4 x 512 lanes; one hot column on top needs owners that do not exist
    m, n, r, d = 8, 2048, 2048, 16
    rng = np.random.default_rng(3)
    P_idx, P_val = syn.ell_projector(m, r, d, rng)
    Q_idx, Q_val = syn.ell_projector(n, r, d, rng, "distinct")
    Q_idx[:, 0] = 0
    nb = L.lsp_plan_bytes(m, n, r, d)
    host = np.zeros(nb, dtype=np.uint8)
    assert L.lsp_plan_build_host(P_idx, P_val, Q_idx, Q_val, m, n, r, d, host, nb, check=False) == -8
    dev = [torch.from_numpy(x).cuda() for x in (P_idx, P_val, Q_idx, Q_val)]
    plan = torch.full((nb,), 0xA5, dtype=torch.uint8, device="cuda")
    assert L.lsp_plan_build(*dev, m, n, r, d, plan, nb, torch.cuda.current_stream(), check=False) == -8
    assert int(plan[:4].view(torch.int32).item()) == 0, "a failed build leaves no plan behind"
    # the raw entry serves such projectors through its scatter form, chosen on the device
    import oracle
    import gpu_util as gu
    G = syn.gaussian_matrix(m, n, 1.0, "bf16", rng)
    pb = syn.Problem("skew", m, n, r, d, "bf16", G, G.copy(), P_idx, P_val, Q_idx, Q_val, np.zeros((r, r), np.float32))
    S_o = oracle.compress(G, "bf16", P_idx, P_val, Q_idx, Q_val, r)
    gu.check_compress(gu.DeviceProblem(pb).compress_raw(), S_o, "raw entry on unplannable projectors", 2e-4)
    # an index outside [0, r)
    bad = dev[2].clone()
    bad[5, 1] = r
    assert L.lsp_plan_build(dev[0], dev[1], bad, dev[3], m, n, r, d, plan, nb, torch.cuda.current_stream(), check=False) == -6
    assert int(plan[:4].view(torch.int32).item()) == 0


@pytest.mark.parametrize("m,n,r,dtype", [(1, 2500, 2048, "bf16"), (8, 2500, 2046, "f32"), (9, 2500, 2048, "f16"), (16, 2500, 2046, "f32"), (17, 2500, 2048, "f16"),
                                         (75, 2500, 2047, "bf16"), (8195, 2000, 2048, "f16")])
def test_raw_entry_on_columns_too_skewed_for_a_plan(m, n, r, dtype):
    """The scatter form by blocks of 8 rows: one row, a whole block, one row more, two blocks and three, ten, and three blocks a workgroup."""
    import gpu_util as gu
    import oracle
    import paper_2406_10181_amd as L
    d = 4
    rng = np.random.default_rng(9000 + m)
    P_idx, P_val = syn.ell_projector(m, r, d, rng)
    Q_idx, Q_val = syn.ell_projector(n, r, d, rng)
    Q_idx[:, 0] = np.arange(n) % 2                                  # two columns take a quarter of the entries
    nb = L.lsp_plan_bytes(m, n, r, d)
    G = syn.gaussian_matrix(m, n, 1.0, dtype, rng)
    pb = syn.Problem("skew", m, n, r, d, dtype, G, G.copy(), P_idx, P_val, Q_idx, Q_val, np.zeros((r, r), np.float32))
    print(f"[case] raw entry, skewed m={m} r={r} {dtype}", flush=True)
    assert L.lsp_plan_build_host(P_idx, P_val, Q_idx, Q_val, m, n, r, d, np.zeros(nb, dtype=np.uint8), nb, check=False) == -8
    S_o = oracle.compress(G, dtype, P_idx, P_val, Q_idx, Q_val, r)
    gu.check_compress(gu.DeviceProblem(pb).compress_raw(), S_o, "raw entry on unplannable projectors", 2e-4)


def test_device_plan_and_compress_with_every_lane_taken_and_one_long_list():
    import torch
    import gpu_util as gu
    import oracle
    import paper_2406_10181_amd as L
    m, n, r, d = 40, 4096, 2048, 8
    pb = syn.make_problem("full", m, n, r, d, "bf16", seed=9100, g_std=1.0, index_dist="distinct")
    rows = [j for j in range(2048, n) if 7 not in pb.Q_idx[j]][:30 - int((pb.Q_idx[2048:] == 7).sum())]
    pb.Q_idx[rows, 0] = 7                                           # 30 entries in the second chunk, where 8 are usual
    print("[case] device plan, every lane taken", flush=True)
    nb = L.lsp_plan_bytes(m, n, r, d)
    host = np.zeros(nb, dtype=np.uint8)
    assert L.lsp_plan_build_host(pb.P_idx, pb.P_val, pb.Q_idx, pb.Q_val, m, n, r, d, host, nb, check=False) == 0
    dp = gu.DeviceProblem(pb)
    S = dp.compress_planned()
    assert np.array_equal(dp.plan.cpu().numpy(), host)
    S_o = oracle.compress(pb.G, "bf16", pb.P_idx, pb.P_val, pb.Q_idx, pb.Q_val, r)
    gu.check_compress(S, S_o, "every lane taken")
