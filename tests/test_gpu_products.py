"""The r x r products of re-projection and fitting at the edges of their tiles: one, two, three and many tiles of K, last tiles of four rows, both sizes of tile, and the gather of fitting beside them."""
import numpy as np
import pytest

import lsp_synth as syn

pytestmark = pytest.mark.gpu


def _dense(idx, val, r):
    out = np.zeros((idx.shape[0], r))
    np.add.at(out, (np.arange(idx.shape[0])[:, None], idx), val.astype(np.float64))
    return out


@pytest.mark.parametrize("r", [2, 4, 28, 30, 32, 33, 36, 64, 68, 97, 100, 132, 1020, 1024, 1027, 1028])
def test_reproject_products(r):
    import torch
    import paper_2406_10181_amd as L
    m, n, d = 150, 90, 2
    print(f"[case] products r={r}", flush=True)
    rng = np.random.default_rng(7000 + r)
    prj = [syn.ell_projector(rows, r, d, rng, "uniform") for rows in (m, m, n, n)]     # P, P_prev, Q, Q_prev
    M = rng.standard_normal((r, r)).astype(np.float32)
    V = (rng.standard_normal((r, r)) ** 2).astype(np.float32)
    P, Pp, Q, Qp = (_dense(*x, r) for x in prj)
    A, B = P.T @ Pp, Qp.T @ Q
    dev = [torch.from_numpy(x).cuda() for pair in prj for x in pair]
    Md, Vd = torch.from_numpy(M).cuda(), torch.from_numpy(V).cuda()
    nb = L.lsp_reproject_state_workspace_bytes(r)
    ws = torch.empty(nb, dtype=torch.uint8, device="cuda")
    L.lsp_reproject_state(*dev, m, n, r, d, Md, Vd, ws, nb, torch.cuda.current_stream())
    torch.cuda.synchronize()
    # fp32: two sums of r products each, the factors A and B rounded once (for V squared, and rounded again), all relative to the sums of magnitudes
    bound = (2 * r + 8) * 2.0 ** -24
    for got, want, size in ((Md, A @ M @ B, abs(A) @ abs(M) @ abs(B)), (Vd, A ** 2 @ V @ B ** 2, A ** 2 @ V @ B ** 2)):
        err = np.abs(got.cpu().numpy() - want)
        assert (err <= bound * size + 1e-30).all(), float((err / (size + 1e-30)).max())


@pytest.mark.parametrize("m,n,r,d,dtype", [
    (70, 24, 4, 1, "f16"),           # one workgroup a product: the gather's first is number 8
    (300, 520, 100, 4, "bf16"),      # 16 tiles of a product, the last four rows and columns wide
    (520, 300, 1028, 2, "f32"),      # 64 x 64 tiles
    (260, 310, 33, 3, "f32"),        # r no multiple of 4: floats one by one
    (64, 6, 36, 2, "bf16"),          # fewer columns than a 16-byte piece of G
])
def test_gradient_with_products_beside_the_gather(m, n, r, d, dtype):
    from test_gpu_fitting import _check_gradient
    _check_gradient(syn.make_problem("products", m, n, r, d, dtype, seed=7100 + r, g_std=1.0, index_dist="uniform"))
