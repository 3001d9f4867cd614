"""Plan build on the device with lanes left over, at the bound below which a share is not split: many columns with lists of 63 pairs, or of 64, or fewer, against the host's owners."""
import numpy as np
import pytest

import lsp_synth as syn

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,r,d,kind,longest,of_64", [
    (2048, 300, 4, "uniform", None, 0),          # no share of 64 among 300 columns
    (2048, 261, 8, "equal", 63, 0),              # none, but by one pair
    (2048, 260, 8, "equal", 64, 4),              # four of 260: most of the lanes stay over
    (2048, 256, 8, "equal", 64, 256),            # every column, and every lane
])
def test_owners_at_the_bound(n, r, d, kind, longest, of_64):
    import torch
    import paper_2406_10181_amd as L
    print(f"[case] spare lanes at the bound n={n} r={r} d={d} {kind}", flush=True)
    m = 40
    rng = np.random.default_rng(8900 + n + r)
    P, Q = (list(syn.ell_projector(rows, r, d, rng, "uniform")) for rows in (m, n))
    if kind == "equal":
        Q[0] = (np.arange(n * d) % r).reshape(n, d).astype(np.int32)
    counts = np.bincount(Q[0].reshape(-1), minlength=r)               # (one chunk)
    assert (longest is None or counts.max() == longest) and (counts >= 64).sum() == of_64
    nb = L.lsp_plan_bytes(m, n, r, d)
    host = np.zeros(nb, np.uint8)
    assert L.lsp_plan_build_host(P[0], P[1], Q[0], Q[1], m, n, r, d, host, nb, check=False) == 0
    dev = [torch.from_numpy(np.ascontiguousarray(x)).cuda() for x in (*P, *Q)]
    plan = torch.full((nb,), 0xA5, dtype=torch.uint8, device="cuda")
    wb = L.lsp_plan_build_workspace_bytes(m, n, r, d)
    ws = torch.empty(wb, dtype=torch.uint8, device="cuda")
    status = torch.full((1,), 77, dtype=torch.int32, device="cuda")
    L.lsp_plan_build_async(*dev, m, n, r, d, plan, nb, ws, wb, status, torch.cuda.current_stream())
    torch.cuda.synchronize()
    assert int(status.item()) == 0
    assert np.array_equal(plan.cpu().numpy(), host)
