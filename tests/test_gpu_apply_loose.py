"""The apply step and the bias pass where rows begin anywhere or d is none of 2, 4, 8, 16 (k_expand_loose), at its edges: columns behind the last whole patch (8 of 16 bits, 4 of
fp32; 4 and 2 in blocks of 8 rows) from none to the most, a pass and a bit, r with a last quad of every length, few rows (m = 13: blocks of 8; in the fp32 apply
step blocks of 4 in the kernel with units of 4), blocks of 16 on one workgroup a CU (2069) and on more (4100), last blocks that are not whole."""
import pytest

import lsp_synth as syn
import oracle


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["bf16", "f16", "f32"])
@pytest.mark.parametrize("m,n,r,d", [
    (13, 1025, 21, 2), (13, 1026, 22, 3), (13, 1031, 23, 7), (13, 2049, 1023, 12), (13, 1028, 16, 5), (1, 1033, 9, 9),
    (2069, 1025, 130, 3), (2069, 1030, 131, 5), (2069, 1039, 260, 11), (2069, 2055, 257, 6), (2065, 301, 50, 9), (2069, 1032, 254, 4), (2070, 4098, 60, 2), (2069, 1026, 66, 8),
    (4100, 1537, 130, 3), (4113, 1543, 67, 10), (4100, 2048, 99, 2), (4100, 1540, 68, 7), (4100, 2050, 262, 8), (8200, 1801, 66, 4), (16390, 1538, 260, 8),
])
def test_apply_and_bias_of_rows_that_begin_anywhere(m, n, r, d, dtype):
    import gpu_util as gu
    from test_gpu_parity import _bias_check
    print(f"[case] loose m={m} n={n} r={r} d={d} {dtype}", flush=True)
    pb = syn.make_problem("loose", m, n, r, d, dtype, seed=9950 + m + n + r + d, g_std=1.0)
    Wp, Wr = oracle.decompress_apply(pb.W, dtype, pb.S_in, pb.P_idx, pb.P_val, pb.Q_idx, pb.Q_val)
    gu.check_decompress(gu.DeviceProblem(pb).decompress(pb.S_in), pb.W, Wp, Wr, dtype, pb.name)
    _bias_check(pb)


# Integers: every sum is exact, so what the kernel makes of each place is the oracle's, bit for bit; elements beside the matrix stay as they were.
@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["bf16", "f16", "f32"])
@pytest.mark.parametrize("m,n,r,d", [(13, 1029, 13, 3), (2069, 1031, 30, 7), (4100, 1543, 17, 5)])
def test_nothing_beside_the_matrix_is_touched(m, n, r, d, dtype):
    import numpy as np
    import torch
    import gpu_util as gu
    import paper_2406_10181_amd as lsp
    rng = np.random.default_rng(m + n)
    t = {"bf16": torch.bfloat16, "f16": torch.float16, "f32": torch.float32}[dtype]
    code = {"f32": 0, "f16": 1, "bf16": 2}[dtype]
    P_idx, Q_idx = (torch.from_numpy(rng.integers(0, r, (k, d), dtype=np.int32)) for k in (m, n))
    P_val, Q_val = (torch.from_numpy(rng.integers(-1, 2, (k, d)).astype(np.float32)) for k in (m, n))
    S = torch.from_numpy(rng.integers(-1, 2, (r, r)).astype(np.float32))
    W = torch.from_numpy(rng.integers(-8, 9, (m, n)).astype(np.float32))
    guard = 64
    all_of_it = torch.full((m * n + guard,), 7.0, dtype=t, device="cuda")
    all_of_it[: m * n] = W.to(t).reshape(-1).cuda()
    lsp.lsp_decompress_apply(all_of_it, S.cuda(), P_idx.cuda(), P_val.cuda(), Q_idx.cuda(), Q_val.cuda(), m, n, r, d, code, torch.cuda.current_stream())
    dense_p, dense_q = (torch.zeros(k, r, dtype=torch.float64).scatter_add_(1, i.long(), v.double()) for k, i, v in ((m, P_idx, P_val), (n, Q_idx, Q_val)))
    want = (W.double() - dense_p @ S.double() @ dense_q.T).to(t)
    got = all_of_it.cpu()
    assert (got[m * n:] == 7.0).all()
    assert torch.equal(got[: m * n].reshape(m, n), want)


def test_every_kernel_is_launched_for_some_shape(tmp_path):
    import os
    import subprocess
    import sys
    from test_launches import ROOT, STAND_IN
    calls = r"""
import ctypes, sys
shim = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
sys.path.insert(0, sys.argv[2])
import paper_2406_10181_amd as L
fake, big = 0x1000, 1 << 40
for r in (16, 1024, 300):
    for m in (300, 2000, 3000, 9000):
        for n in (301, 4099):
            for d in range(1, 17):
                for code in (0, 1, 2):
                    L.lsp_decompress_apply(fake, fake, fake, fake, fake, fake, m, n, r, d, code)
                    L.lsp_estimation_bias(fake, fake, fake, fake, fake, fake, m, n, r, d, fake, fake, big, code)
shim.launches_beyond.restype = ctypes.c_long
print("beyond", shim.launches_beyond())
shim.print_never_launched(b"k_expand_loose")
sys.stdout.flush()
"""
    src, so = tmp_path / "stand_in.cpp", tmp_path / "stand_in.so"
    src.write_text(STAND_IN)
    subprocess.run([os.environ.get("CXX", "g++"), "-O1", "-std=c++17", "-shared", "-fPIC", str(src), "-o", str(so)], check=True)
    out = subprocess.run([sys.executable, "-c", calls, str(so), ROOT], capture_output=True, text=True, timeout=300)
    assert out.returncode == 0 and "beyond 0" in out.stdout and "never launched" not in out.stdout, (out.stdout[-2000:], out.stderr[-2000:])


# The apply step with few rows: blocks of 4 (and of 8: d = 16, and 16 bits with odd rows) whose passes are shared by up to as many workgroups as there are passes; both sides of the rule
# (64 and 65 blocks of 16 rows; fp32 112, 113, 128 and 129).
@pytest.mark.gpu
@pytest.mark.parametrize("m,n,r,d,dtype", [
    (m, n, r, d, dtype) for dtype in ("bf16", "f16", "f32")
    for m, n, r, d in [(1, 8, 4, 2), (3, 2056, 16, 4), (5, 4104, 260, 8), (255, 1024, 300, 8), (257, 3080, 700, 2), (1024, 1032, 128, 4), (1025, 1032, 128, 4), (16, 5128, 20, 16),
                       (130, 3072, 600, 16), (7, 3077, 31, 5), (129, 2051, 300, 13), (66, 4099, 50, 1), (40, 2050, 1000, 8), (33, 6151, 90, 12)]
] + [(1792, 520, 60, 4, "f32"), (1793, 520, 60, 4, "f32"), (2048, 1032, 260, 8, "f32"), (2049, 520, 600, 2, "f32"), (2048, 520, 516, 4, "f32")])
def test_apply_with_few_rows(m, n, r, d, dtype):
    import torch
    import gpu_util as gu
    import paper_2406_10181_amd as lsp
    print(f"[case] few rows m={m} n={n} r={r} d={d} {dtype}", flush=True)
    pb = syn.make_problem("few rows", m, n, r, d, dtype, seed=9970 + m + n + r + d, g_std=1.0)
    Wp, Wr = oracle.decompress_apply(pb.W, dtype, pb.S_in, pb.P_idx, pb.P_val, pb.Q_idx, pb.Q_val)
    dp = gu.DeviceProblem(pb)
    single = dp.decompress(pb.S_in)
    gu.check_decompress(single, pb.W, Wp, Wr, dtype, pb.name)
    # in a group with a larger matrix other kernels make the same bits
    other = gu.DeviceProblem(syn.make_problem("larger", 2100, 40, r, d, dtype, seed=2, g_std=1.0))
    dp.W.copy_(gu.to_device(pb.W, dtype))
    S = gu.to_device(pb.S_in)
    items = [(x.W, S, x.P_idx, x.P_val, x.Q_idx, x.Q_val, x.pb.m, x.pb.n) for x in (dp, other)]
    lsp.lsp_decompress_apply_grouped(lsp.apply_items(items), 2, r, d, dp.code, torch.cuda.current_stream())
    torch.cuda.synchronize()
    assert (gu.to_host(dp.W, dtype) == single).all()
