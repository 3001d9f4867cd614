"""Kernel A for bf16 (compress_mm.hip) at the edges of its tiles, rows, chunks and of the LDS, against 64-bit sums: random values with full
mantissas, and matrices with infinities and NaN."""
import numpy as np
import pytest

import lsp_synth as syn

pytestmark = pytest.mark.gpu


def _problem(m, n, r, seed, dist, d=1):
    """d entries a row of Q; row i of P names column i % r, with value one (and zeros in further entries).  dist "hot": nearly all entries of a
    chunk are in one column, another one in every chunk, so that there are many more lists than columns."""
    rng = np.random.default_rng(seed)
    Q_idx, Q_val = syn.ell_projector(n, r, d, rng, "uniform" if dist == "hot" else dist)
    if dist == "hot":
        rows = np.flatnonzero(rng.random(n) < 0.95)
        Q_idx[rows] = (rows // 2048 % r)[:, None]
    P_idx = np.repeat((np.arange(m, dtype=np.int32) % r)[:, None], d, axis=1).copy()
    P_val = np.zeros((m, d), np.float32)
    P_val[:, 0] = 1.0
    G = syn.to_storage(rng.standard_normal((m, n)).astype(np.float32), "bf16")
    return syn.Problem("mm", m, n, r, d, "bf16", G, G.copy(), P_idx, P_val, Q_idx, Q_val, np.zeros((r, r), np.float32))


def _exact(pb):
    """S, the sums of the magnitudes, and the terms of the longest sum."""
    G = syn.storage_to_f64(pb.G, "bf16")
    T, A = np.zeros((pb.m, pb.r)), np.zeros((pb.m, pb.r))
    with np.errstate(invalid="ignore"):
        for k in range(pb.d):
            GQ = G * pb.Q_val[:, k].astype(np.float64)
            np.add.at(T.T, pb.Q_idx[:, k], GQ.T)
            np.add.at(A.T, pb.Q_idx[:, k], np.abs(GQ).T)
        S, B = np.zeros((pb.r, pb.r)), np.zeros((pb.r, pb.r))
        np.add.at(S, pb.P_idx[:, 0], T)
        np.add.at(B, pb.P_idx[:, 0], A)
    terms = np.bincount(pb.Q_idx.reshape(-1)).max() + np.bincount(pb.P_idx.reshape(-1)).max()
    return S, B, int(terms)


SHAPES = [
    (1, 5, 3, "uniform"), (3, 8, 1, "uniform"),                   # fewer columns than a piece of G; one list
    (4, 9, 40, "uniform"), (8, 2047, 31, "uniform"),              # a piece that ends before the row; a chunk less one
    (9, 2049, 33, "uniform"), (17, 4103, 250, "uniform"),         # a second row block; a last chunk of one and of seven columns
    (16, 6144, 512, "uniform"), (33, 4100, 1100, "uniform"),      # 16 whole tiles; more than 1024 columns
    (40, 2500, 2048, "uniform"), (50, 4096, 20, "zipf"),          # all tiles of a wave; shared columns
    (2048, 264, 48, "uniform"), (2049, 264, 48, "zipf"),          # the last with blocks of 8 rows, the first with blocks of 16
    (4081, 520, 64, "uniform"), (4096, 2056, 96, "zipf"),         # one 16-row block a workgroup
    (4097, 300, 33, "uniform"), (6144, 67, 33, "uniform"),        # three rounds of 8-row blocks, where those of 16 would take two: the first rows and the last
    (6145, 67, 33, "uniform"), (6544, 67, 33, "uniform"),         # two rounds of 16-row blocks, a little over half full
    (6545, 67, 33, "uniform"), (8192, 264, 48, "zipf"),           # two 16-row blocks a workgroup, not for all and for all; n % 8 != 0
    (4096, 300, 1024, "uniform"), (4096, 2100, 1024, "zipf"),     # the most columns 16-row blocks are used for; some of them shared
    (2061, 10245, 1024, "hot"),                                   # more than 1376 lists: the sums of 16 rows do not fit the LDS, blocks go in halves
]


@pytest.mark.parametrize("m,n,r,dist", SHAPES)
def test_bf16_compress_at_the_edges(m, n, r, dist):
    import gpu_util as gu
    pb = _problem(m, n, r, 7000 + m + n + r, dist)
    print(f"[case] mm m={m} n={n} r={r} {dist}", flush=True)
    S, B, terms = _exact(pb)
    got = gu.DeviceProblem(pb).compress_planned().astype(np.float64)
    # every term passes at most `terms` additions in fp32, and a product of the split values is exact but for the adding of its parts
    assert (np.abs(got - S) <= (terms + 4) * 2.0 ** -24 * B + 1e-35).all(), (np.abs(got - S) / (B + 1e-30)).max() * 2 ** 24


@pytest.mark.parametrize("m,n,r,dist", [(17, 4103, 250, "uniform"), (9, 2049, 33, "uniform"), (4096, 2056, 96, "zipf"), (40, 2500, 2048, "uniform")])
def test_bf16_compress_with_infinities_and_nan(m, n, r, dist):
    """Only the sums that an infinity or a NaN belongs to may notice: neither the zeros that fill up a tile nor the lower parts of a value."""
    import gpu_util as gu
    pb = _problem(m, n, r, 7100 + m + n + r, dist)
    rng = np.random.default_rng(m)
    for bits in (0x7F80, 0xFF80, 0x7FC0):
        for _ in range(3):
            pb.G[rng.integers(m), rng.integers(n)] = bits
    pb.G[rng.integers(m), 0] = 0x7F80
    pb.G[m - 1, n - 1] = 0xFF80
    print(f"[case] mm inf m={m} n={n} r={r} {dist}", flush=True)
    S, B, terms = _exact(pb)
    got = gu.DeviceProblem(pb).compress_planned().astype(np.float64)
    finite = np.isfinite(S)
    assert np.array_equal(np.isfinite(got), finite)
    assert (np.abs(got[finite] - S[finite]) <= (terms + 4) * 2.0 ** -24 * B[finite] + 1e-35).all()


@pytest.mark.parametrize("m,n,r", [(40, 2500, 2048), (4096, 300, 1024)])
def test_bf16_compress_keeps_infinities_and_their_signs(m, n, r):
    """Blocks of 8 rows and of 16, and as many rows in every row of P^T as kernel B takes at a time, so that it adds no zeros: an infinity stays
    one, and only sums of both infinities, or with a NaN, are NaN."""
    import gpu_util as gu
    pb = _problem(m, n, r, 7150 + m, "uniform")
    rng = np.random.default_rng(m)
    for bits in (0x7F80, 0xFF80, 0x7FC0):
        for _ in range(40):
            pb.G[rng.integers(m), rng.integers(n)] = bits
    pb.Q_val[:40] = np.float32(0.5)                                   # (lower parts that are zero)
    pb.G[m - 1, :40] = 0x7F80
    print(f"[case] mm signs of infinities m={m} n={n} r={r}", flush=True)
    S, _, _ = _exact(pb)
    got = gu.DeviceProblem(pb).compress_planned().astype(np.float64)
    for kind in (np.isposinf, np.isneginf, np.isnan):
        assert kind(S).any() and np.array_equal(kind(got), kind(S)), kind.__name__


def test_bf16_compress_that_overflows_is_infinite():
    """The largest bf16 number times values whose first part is one: only the lower parts take the product beyond fp32."""
    import gpu_util as gu
    m, n, r = 40, 600, 2048
    pb = _problem(m, n, r, 7160, "uniform")
    pb.Q_idx[:, 0] = np.arange(n)
    pb.Q_val[:, 0] = np.where(np.arange(n) % 2, np.float32(1.0077), np.float32(1.0))
    pb.G[:] = np.where(np.arange(m)[:, None] % 3 == 0, 0xFF7F, 0x7F7F)
    print("[case] mm overflow", flush=True)
    got = gu.DeviceProblem(pb).compress_planned()
    with np.errstate(over="ignore"):
        want = (syn.storage_to_f64(pb.G, "bf16") * pb.Q_val[:, 0].astype(np.float64)).astype(np.float32)
    assert np.isinf(want).any() and np.isfinite(want).any()
    assert np.array_equal(got[:m, :n], want) and not got[m:].any() and not got[:, n:].any()


@pytest.mark.parametrize("m,n,r,d,dist", [(2049, 520, 64, 8, "uniform"), (33, 4103, 512, 16, "zipf"), (50, 2500, 2048, 4, "uniform"), (4100, 264, 96, 3, "zipf")])
def test_bf16_compress_with_several_entries_a_row(m, n, r, d, dist):
    import gpu_util as gu
    pb = _problem(m, n, r, 7200 + m + n + r, dist, d)
    print(f"[case] mm m={m} n={n} r={r} d={d} {dist}", flush=True)
    S, B, terms = _exact(pb)
    got = gu.DeviceProblem(pb).compress_planned().astype(np.float64)
    assert (np.abs(got - S) <= (terms + 4) * 2.0 ** -24 * B + 1e-35).all(), (np.abs(got - S) / (B + 1e-30)).max() * 2 ** 24


def _group(dps, r, d, plans=None):
    """S of a grouped call, each filled with ones before."""
    import torch
    import paper_2406_10181_amd as L
    for dp in dps:
        dp.S.fill_(1.0)
    items = L.compress_items([(dp.G, plans[k] if plans and k in plans else dp.plan, dp.S, dp.ws, dp.ws_bytes, dp.pb.m, dp.pb.n) for k, dp in enumerate(dps)])
    L.lsp_compress_planned_grouped(items, len(dps), r, d, 2, torch.cuda.current_stream())
    torch.cuda.synchronize()
    return [dp.S.cpu().numpy() for dp in dps]


@pytest.mark.parametrize("shapes,r,d", [
    ([(5120, 264, "uniform")] * 2, 48, 1),                                           # 8-row blocks alone, three rounds of 16-row blocks together
    ([(2500, 264, "uniform"), (2600, 300, "zipf")], 96, 4),                          # 16-row blocks alone, three rounds of 8-row blocks together
    ([(5120, 2056, "zipf"), (2112, 264, "uniform"), (2112, 2050, "uniform")], 512, 8),   # a round of 8-row blocks each; n % 8 != 0 for one
    ([(40, 2500, "uniform"), (2048, 264, "uniform"), (4096, 300, "uniform")], 1024, 2),   # 8-row blocks alone, 16-row blocks together
    ([(300, 520, "uniform"), (1001, 10240, "hot"), (4096, 264, "uniform")], 1024, 1),    # sums of 16 rows that fit the LDS, and some that go in halves
    ([(300, 520, "uniform"), (17, 4103, "uniform")], 2048, 3),                       # 8-row blocks throughout
])
def test_bf16_compress_in_a_group_is_that_of_the_single_calls(shapes, r, d):
    import gpu_util as gu
    print(f"[case] mm group {shapes} r={r} d={d}", flush=True)
    dps = [gu.DeviceProblem(_problem(m, n, r, 7300 + k + m + n, dist, d)) for k, (m, n, dist) in enumerate(shapes)]
    singles = [dp.compress_planned() for dp in dps]
    for single, grouped in zip(singles, _group(dps, r, d)):
        assert np.isfinite(single).all() and np.array_equal(single, grouped), np.abs(single - grouped).max()


# More than two chunks: blocks begin with different ones.  Two blocks in halves for a workgroup; two chunks in LDS at a time, with one block a workgroup, two, and blocks of 8 rows.
@pytest.mark.parametrize("m,n,r,dist", [(6160, 6150, 1024, "hot"), (6545, 6151, 33, "uniform"), (2500, 8195, 33, "uniform"), (300, 8195, 250, "zipf"), (520, 6152, 512, "uniform")])
def test_bf16_compress_over_many_chunks(m, n, r, dist):
    test_bf16_compress_at_the_edges(m, n, r, dist)


# The same rows in blocks of 8 and of 16, and beside matrices whose sums leave no room for two chunks.
@pytest.mark.parametrize("shapes,r,d", [
    ([(5120, 6152, "uniform")] * 2, 48, 1),
    ([(2500, 8200, "uniform"), (2600, 6150, "zipf")], 96, 4),
    ([(40, 6150, "uniform"), (2048, 8192, "uniform"), (4096, 6152, "zipf")], 1000, 2),
    ([(300, 6152, "uniform"), (2500, 10240, "hot"), (4096, 264, "uniform")], 320, 1),
])
def test_bf16_compress_over_many_chunks_in_a_group(shapes, r, d):
    test_bf16_compress_in_a_group_is_that_of_the_single_calls(shapes, r, d)


@pytest.mark.parametrize("foreign", [0, 1, 2])
def test_bf16_compress_with_a_foreign_plan_in_a_group(foreign):
    """Its S is NaN and its workspace untouched; the others are served as if it were not there."""
    import torch
    import gpu_util as gu
    r, d = 64, 2
    shapes = [(300, 4100), (4096, 520), (2049, 264)]
    print(f"[case] mm group, plan {foreign} is foreign", flush=True)
    dps = [gu.DeviceProblem(_problem(m, n, r, 7400 + m, "uniform", d)) for m, n in shapes]
    singles = [dp.compress_planned() for dp in dps]
    m, n = shapes[foreign]
    other = gu.DeviceProblem(_problem(m + 8, n, r, 7500, "uniform", d))
    other.build_plan()
    dps[foreign].ws.fill_(0x5A)
    grouped = _group(dps, r, d, {foreign: other.plan})
    for k in range(3):
        if k == foreign:
            assert np.isnan(grouped[k]).all() and bool((dps[k].ws == 0x5A).all())
        else:
            assert np.array_equal(singles[k], grouped[k])


@pytest.mark.parametrize("kind,r,dtype", [("older layout", 64, "bf16"), ("older layout", 3, "bf16"), ("older layout", 64, "f16"), ("older layout", 64, "f32"),
                                          ("no tiles", 64, "bf16"), ("no tiles", 3, "bf16")])
def test_compress_refuses_a_plan_it_cannot_follow(kind, r, dtype):
    """A plan of this very problem, but of an older layout, or the one that a raw call makes in its workspace, which has no tiles: S is NaN
    throughout (kernel B may not put sums over what lies in T in its place) and T is untouched."""
    import torch
    import gpu_util as gu
    import paper_2406_10181_amd as L
    pb = syn.make_problem("refused", 300, 2100, r, 2, dtype, seed=7550 + r, g_std=1.0)
    print(f"[case] plan refused: {kind} r={r} {dtype}", flush=True)
    dp = gu.DeviceProblem(pb)
    dp.build_plan()
    if kind == "older layout":
        dp.plan[:4].view(torch.int32).fill_(0x4C535038)
    else:
        dp.compress_raw()
        at = (pb.m * r * 4 + 255) // 256 * 256
        dp.plan = dp.ws[at:at + dp.plan_bytes].clone()
        assert dp.plan[:4].view(torch.int32).item() == 0x4C535039, "the plan of the raw call"
    dp.ws.fill_(0x5A)
    dp.S.fill_(1.0)
    L.lsp_compress_planned(dp.G, dp.plan, pb.m, pb.n, r, 2, dp.S, dp.code, dp.ws, dp.ws_bytes, torch.cuda.current_stream())
    torch.cuda.synchronize()
    assert bool(dp.S.isnan().all()) and bool((dp.ws == 0x5A).all())


@pytest.mark.parametrize("g_exp,v_exp", [
    (0, -100), (60, -118), (60, -124),        # values whose lower parts, as they are, would be subnormal or gone
    (100, -132), (100, -140),                 # subnormal values
    (-126, 60), (-133, 40),                   # gradients partly and all subnormal
    (-126, 0), (-130, 2), (-60, -60), (-64, -75),   # sums that are subnormal in fp32, in part and all
    (120, 0), (64, 55),                       # sums near the largest number
])
def test_bf16_compress_at_the_ends_of_the_exponents(g_exp, v_exp):
    import gpu_util as gu
    pb = _problem(40, 2500, 96, 7600, "uniform")
    rng = np.random.default_rng(7600 - g_exp)
    G = np.ldexp(rng.uniform(0.5, 2.0, (pb.m, pb.n)) * rng.choice([-1.0, 1.0], (pb.m, pb.n)), g_exp)
    pb.G = syn.to_storage(G.astype(np.float32), "bf16")
    pb.Q_val = np.ldexp(rng.uniform(0.5, 2.0, pb.Q_val.shape) * rng.choice([-1.0, 1.0], pb.Q_val.shape), v_exp).astype(np.float32)
    print(f"[case] mm exponents {g_exp} {v_exp}", flush=True)
    S, B, terms = _exact(pb)
    assert np.abs(S).max() > 0 and B.max() < 2.0 ** 127
    got = gu.DeviceProblem(pb).compress_planned().astype(np.float64)
    # half a unit in the last place for every addition and for adding the parts, and where sums are subnormal that is 2^-150 at the least;
    # the stored parts leave out a last bit of 2^-149 of values below 2^-125
    lost = 2.0 ** -149 * np.abs(syn.storage_to_f64(pb.G, "bf16")).max() * terms if v_exp < -124 else 0.0
    bound = (terms + 4) * (2.0 ** -24 * B + 2.0 ** -150) + lost
    assert (np.abs(got - S) <= bound).all(), (np.abs(got - S) / bound).max()
