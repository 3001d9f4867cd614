"""Kernel A for bf16 (compress_mm.hip) at the edges of its tiles, rows, chunks and of the LDS, against 64-bit sums: random values with full
mantissas, and matrices with infinities and NaN."""
import numpy as np
import pytest

import lsp_synth as syn

pytestmark = pytest.mark.gpu


def _problem(m, n, r, seed, dist):
    """One entry a row; row i of P names column i % r, with value one."""
    rng = np.random.default_rng(seed)
    Q_idx, Q_val = syn.ell_projector(n, r, 1, rng, dist)
    P_idx = (np.arange(m, dtype=np.int32) % r)[:, None].copy()
    P_val = np.ones((m, 1), np.float32)
    G = syn.to_storage(rng.standard_normal((m, n)).astype(np.float32), "bf16")
    return syn.Problem("mm", m, n, r, 1, "bf16", G, G.copy(), P_idx, P_val, Q_idx, Q_val, np.zeros((r, r), np.float32))


def _exact(pb):
    """S, the sums of the magnitudes, and the terms of the longest sum."""
    G = syn.storage_to_f64(pb.G, "bf16")
    T, A = np.zeros((pb.m, pb.r)), np.zeros((pb.m, pb.r))
    with np.errstate(invalid="ignore"):
        GQ = G * pb.Q_val[:, 0].astype(np.float64)
        np.add.at(T.T, pb.Q_idx[:, 0], GQ.T)
        np.add.at(A.T, pb.Q_idx[:, 0], np.abs(GQ).T)
        S, B = np.zeros((pb.r, pb.r)), np.zeros((pb.r, pb.r))
        np.add.at(S, pb.P_idx[:, 0], T)
        np.add.at(B, pb.P_idx[:, 0], A)
    terms = np.bincount(pb.Q_idx[:, 0]).max() + np.bincount(pb.P_idx[:, 0]).max()
    return S, B, int(terms)


SHAPES = [
    (1, 5, 3, "uniform"), (3, 8, 1, "uniform"),                   # fewer columns than a piece of G; one list
    (4, 9, 40, "uniform"), (8, 2047, 31, "uniform"),              # a piece that ends before the row; a chunk less one
    (9, 2049, 33, "uniform"), (17, 4103, 250, "uniform"),         # a second row block; a last chunk of one and of seven columns
    (16, 6144, 512, "uniform"), (33, 4100, 1100, "uniform"),      # 16 whole tiles; more than 1024 columns
    (40, 2500, 2048, "uniform"), (50, 4096, 20, "zipf"),          # all tiles of a wave; shared columns
    (2048, 264, 48, "uniform"), (2049, 264, 48, "zipf"),          # the last with blocks of 8 rows, the first with blocks of 16
    (4081, 520, 64, "uniform"), (4096, 2056, 96, "zipf"),         # one 16-row block a workgroup
    (4097, 300, 33, "uniform"), (6544, 67, 33, "uniform"),        # k_compress_gq takes these: the last round is too empty
    (6545, 67, 33, "uniform"), (8192, 264, 48, "zipf"),           # two 16-row blocks a workgroup, not for all and for all; n % 8 != 0
    (4096, 300, 1024, "uniform"), (4096, 2100, 1024, "zipf"),     # the most columns 16-row blocks are used for; more sums than the LDS holds
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
