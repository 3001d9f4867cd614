"""Kernel B of compress (S = P^T T) keeps infinities and their signs whatever the lengths of the rows of P^T: groups of lanes that have no entry in a piece's last step add zeros,
and not zero times a row of T."""
import numpy as np
import pytest

import lsp_synth as syn

pytestmark = pytest.mark.gpu


def _problem(m, n, r, dtype, seed):
    """One entry a row of P and of Q; a third of the rows of G has an infinity."""
    rng = np.random.default_rng(seed)
    P_idx, Q_idx = (rng.integers(0, r, (k, 1), dtype=np.int32) for k in (m, n))
    P_idx[:r, 0] = np.arange(r)[:m]                                   # every row of P^T has an entry
    P_val, Q_val = np.ones((m, 1), np.float32), np.full((n, 1), 0.5, np.float32)
    G = rng.standard_normal((m, n)).astype(np.float32)
    rows = np.flatnonzero(rng.random(m) < 1 / 3)
    G[rows, rng.integers(0, n, rows.size)] = np.where(rng.random(rows.size) < 0.5, np.inf, -np.inf)
    G = syn.to_storage(G, dtype)
    return syn.Problem("infinities", m, n, r, 1, dtype, G, G.copy(), P_idx, P_val, Q_idx, Q_val, np.zeros((r, r), np.float32))


@pytest.mark.parametrize("m,n,r,dtype", [
    (64, 24, 33, "f32"), (1200, 12, 16, "f16"), (300, 40, 64, "bf16"), (1400, 24, 250, "f32"), (1500, 24, 256, "bf16"),   # eight groups of lanes
    (1500, 24, 260, "f32"), (2500, 24, 512, "bf16"), (2500, 33, 511, "f16"),                                             # four
    (2600, 24, 600, "f16"), (4100, 24, 1024, "bf16"),                                                                     # two
    (4100, 24, 2000, "bf16"),                                                                                             # one
    (6000, 24, 2047, "f16"),
    (9000, 24, 2048, "f32"), (8400, 24, 2048, "bf16"),                                                                    # two rounds: two groups
    (8400, 24, 1024, "f16"),                                                                                              # four
])
def test_infinities_and_their_signs(m, n, r, dtype):
    import gpu_util as gu
    print(f"[case] infinities m={m} n={n} r={r} {dtype}", flush=True)
    pb = _problem(m, n, r, dtype, 6600 + m + r)
    G = syn.storage_to_f64(pb.G, dtype)
    S, B = np.zeros((r, r)), np.zeros((r, r))
    with np.errstate(invalid="ignore"):
        at = (np.broadcast_to(pb.P_idx, (m, n)), np.broadcast_to(pb.Q_idx.T, (m, n)))
        np.add.at(S, at, 0.5 * G)
        np.add.at(B, at, np.abs(0.5 * G))
    got = gu.DeviceProblem(pb).compress_planned().astype(np.float64)
    for kind in (np.isposinf, np.isneginf, np.isnan):
        assert np.array_equal(kind(got), kind(S)), (kind.__name__, int(kind(got).sum()), int(kind(S).sum()))
    assert np.isposinf(S).any() and np.isneginf(S).any()
    finite = np.isfinite(S)
    terms = np.bincount(pb.P_idx[:, 0]).max() * np.bincount(pb.Q_idx[:, 0]).max()   # every term passes at most that many additions in fp32
    assert (np.abs(got[finite] - S[finite]) <= (terms + 4) * 2.0 ** -24 * B[finite] + 1e-35).all()
