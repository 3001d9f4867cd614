"""Plan build on the device with lanes left over (r < 512): the owners that the search gives out against the host's, one at a time."""
import numpy as np
import pytest

import lsp_synth as syn

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,r,d,kind", [
    (4096, 256, 8, "uniform"),      # nearly every column once more
    (2048, 511, 64, "uniform"),     # one lane left over
    (2048, 400, 16, "equal"),       # all shares equal: 112 of 400 columns, the lowest
    (2100, 448, 32, "equal"),       # two levels, the lower one in the short last chunk
    (4096, 500, 16, "uniform"),     # few lanes, shares on both sides of the level
    (3000, 100, 64, "steps"),       # shares of many kinds, several lanes a column
    (4096, 64, 64, "one"),          # one column has half of all
    (2048, 300, 8, "uniform"),      # few shares of 64 and more (38 of 300)
    (70, 1, 1, "uniform"),          # a list of 70 to share
    (63, 1, 1, "uniform"),          # and one too short
])
def test_owners_as_on_the_host(n, r, d, kind):
    import torch
    import paper_2406_10181_amd as L
    print(f"[case] spare lanes n={n} r={r} d={d} {kind}", flush=True)
    m = 40
    rng = np.random.default_rng(8800 + n + r)
    P, Q = (list(syn.ell_projector(rows, r, d, rng, "uniform")) for rows in (m, n))
    if kind == "equal":
        Q[0] = (np.arange(n * d) % r).reshape(n, d).astype(np.int32)
    elif kind == "steps":
        Q[0] = np.minimum(r - 1, (r * rng.random((n, d)) ** 2).astype(np.int32) // 10 * 10 + rng.integers(0, 2, (n, d))).astype(np.int32)
    elif kind == "one":
        Q[0][:, ::2] = 3
    nb = L.lsp_plan_bytes(m, n, r, d)
    host = np.zeros(nb, np.uint8)
    rc = L.lsp_plan_build_host(P[0], P[1], Q[0], Q[1], m, n, r, d, host, nb, check=False)
    dev = [torch.from_numpy(np.ascontiguousarray(x)).cuda() for x in (*P, *Q)]
    plan = torch.full((nb,), 0xA5, dtype=torch.uint8, device="cuda")
    wb = L.lsp_plan_build_workspace_bytes(m, n, r, d)
    ws = torch.empty(wb, dtype=torch.uint8, device="cuda")
    status = torch.full((1,), 77, dtype=torch.int32, device="cuda")
    L.lsp_plan_build_async(*dev, m, n, r, d, plan, nb, ws, wb, status, torch.cuda.current_stream())
    torch.cuda.synchronize()
    assert rc == 0 and int(status.item()) == 0
    assert np.array_equal(plan.cpu().numpy(), host)
