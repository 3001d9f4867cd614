"""The work that a program using this library has it do, as cases that can be timed.

Every case is one pass of a piece of LSP-Offload's loop (Alg. 1, Alg. 3) through the public entry points of
`paper_2406_10181_amd`, with everything the program keeps between passes (projectors, plans, workspaces, item
arrays of grouped calls) made beforehand in `prepare`:

  step      per-step work: S = P^T G Q (planned), then W -= P S' Q^T with the update that came back from the CPU
  compress  the first half alone (gradients leave while the backward pass still runs)
  apply     the second half alone
  raw       compress from ELL arrays without a plan (projectors used only once)
  check     MaybeUpdate's test: compress, then the estimation bias of Def. 2
  fit       one iteration of projector fitting: new values into the plan, then the gradient of Eq. 2's data term
  refresh   a change of projectors: plan build, re-projection of the optimiser state, first compress with the plan

A case with count > 1 has that many matrices of alternating shape (m x n, n x m), served by the grouped calls;
"layer" is the seven matrices of a 6.7B-style decoder layer.
"""
from __future__ import annotations

import math

import torch

import lsp_synth as syn
import paper_2406_10181_amd as lsp

_TORCH = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}
_SIZE = {"f32": 4, "f16": 2, "bf16": 2}
_CODE = {"f32": 0, "f16": 1, "bf16": 2}


def _case(name, op, m, n, r, d, dtype, dist="uniform", count=1, heavy=False, reorder=False, layer=False):
    c = {"op": op, "m": m, "n": n, "r": r, "d": d, "dtype": dtype, "dist": dist, "count": count,
         "heavy": heavy, "reorder": reorder, "layer": layer}
    return dict(c, name=name) if name else c


def listed():
    return [
        # configuration 1: one small layer in fp32; three launches, so latency and host work are what counts
        _case("step_small_f32", "step", 256, 256, 16, 2, "f32", "distinct"),
        # configuration 2: an attention projection of a 1.3B-style model
        _case("step_attention_f16", "step", 2048, 2048, 256, 4, "f16"),
        # configuration 3: the MLP pair of a 1.3B-style layer, 1 % of the gradient rows 100 times larger
        _case("step_mlp_pair_f16", "step", 2048, 8192, 512, 4, "f16", count=2, heavy=True),
        # configuration 4, the flagship: all seven matrices of a 6.7B-style layer in one grouped call per direction
        _case("step_layer_bf16", "step", 4096, 11008, 512, 8, "bf16", count=7, reorder=True, layer=True),
        # configuration 5: wide matrix, skewed projector columns, each direction by itself
        _case("compress_wide_zipf_bf16", "compress", 4096, 16384, 512, 8, "bf16", "zipf"),
        _case("apply_wide_zipf_bf16", "apply", 4096, 16384, 1024, 16, "bf16", "zipf"),
        # full-precision training of a 4096-wide projection
        _case("step_square_f32", "step", 4096, 4096, 512, 8, "f32"),
        # the paper's own subspace size on 4096-wide layers
        _case("step_r2048_bf16", "step", 4096, 4096, 2048, 8, "bf16"),
        # nothing divides anything: odd rows, odd columns, r and d off the usual steps
        _case("step_ragged_bf16", "step", 3001, 2999, 250, 5, "bf16"),
        # projectors used once: no plan kept
        _case("raw_square_bf16", "raw", 4096, 4096, 512, 8, "bf16"),
        # MaybeUpdate on a 4096-wide projection: one iteration of fitting ...
        _case("fit_square_bf16", "fit", 4096, 4096, 512, 8, "bf16"),
        # ... and the change of projectors of a wide matrix at the end of it
        _case("refresh_wide_bf16", "refresh", 4096, 11008, 512, 8, "bf16"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["step"] * 8 + ["compress"] * 2 + ["apply"] * 2 + ["raw", "check", "check", "fit", "refresh"])
    dtype = rng.choice(["bf16", "bf16", "f16", "f32"])
    dist = rng.choice(["uniform", "uniform", "uniform", "zipf"])
    ragged = rng.random() < 0.25                       # sizes that divide by nothing in particular
    heavy_op = op in ("fit", "refresh")                # dense r x r products among them
    most = 1 << 24 if ragged or heavy_op else 1 << 26  # elements of one call's matrices
    d = rng.choice([2, 4, 4, 8, 8, 8, 16]) if not ragged else rng.randint(1, 12)
    while True:
        # weight matrices: the short side from a small layer's to a large one's, up to four times as long; the subspace
        # a half to a sixteenth of the short side, as in the configurations
        short = _log_int(rng, 256, 8192)
        long = min(16384, int(short * math.exp(rng.uniform(0.0, math.log(4.0)))))
        r = max(16, min(1024 if dist == "zipf" or heavy_op else 2048, _log_int(rng, short / 16, short / 2)))
        if not ragged:
            short, long, r = short // 64 * 64, long // 64 * 64, r // 16 * 16
        m, n = (short, long) if rng.random() < 0.5 else (long, short)
        count = rng.choice([1, 1, 2, 4, 7]) if op in ("step", "compress", "apply") else 1
        if m * n * count <= most:
            break
    return _case(None, op, m, n, r, d, dtype, dist, count, heavy=rng.random() < 0.2, reorder=rng.random() < 0.5)


def _shapes(c):
    if c["layer"]:
        return [(m, n) for _, m, n in syn.LAYER_67B]
    return [(c["m"], c["n"]) if k % 2 == 0 else (c["n"], c["m"]) for k in range(c["count"])]


def _projector(rows, r, d, dist, gen):
    """Random (d, r)-sparse projector in ELL layout, drawn on the GPU: columns i.i.d. uniform, without replacement,
    or Zipf(1.1) with the hot columns first; values N(0, 1/d)."""
    if dist == "distinct":
        idx = torch.rand(rows, r, device="cuda", generator=gen).argsort(dim=1)[:, :d]
    elif dist == "zipf":
        w = torch.arange(1, r + 1, device="cuda", dtype=torch.float64) ** -1.1
        cdf = torch.cumsum(w, 0) / w.sum()
        idx = torch.searchsorted(cdf, torch.rand(rows, d, device="cuda", generator=gen, dtype=torch.float64)).clamp_(max=r - 1)
    else:
        idx = torch.randint(0, r, (rows, d), device="cuda", generator=gen)
    val = torch.randn(rows, d, device="cuda", generator=gen) / math.sqrt(d)
    return idx.to(torch.int32).contiguous(), val.contiguous()


def _bytes(k):
    return torch.empty(max(int(k), 256), dtype=torch.uint8, device="cuda")


class _Matrix:
    """One weight matrix with what a training program keeps for it."""

    def __init__(self, c, m, n, gen):
        r, d, op, t = c["r"], c["d"], c["op"], _TORCH[c["dtype"]]
        self.m, self.n = m, n
        stream = torch.cuda.current_stream()
        self.P = _projector(m, r, d, c["dist"], gen)
        self.Q = _projector(n, r, d, c["dist"], gen)
        self.Qx = self.Q
        if op != "apply":
            G = torch.randn(m, n, device="cuda", generator=gen) * 1e-3
            if c["heavy"]:
                G[torch.randperm(m, device="cuda", generator=gen)[: max(1, m // 100)]] *= 100.0
            self.G = G.to(t)
            self.S = torch.empty(r, r, device="cuda")
        if op in ("step", "apply"):
            self.W = (torch.randn(m, n, device="cuda", generator=gen) * 0.02).to(t)
            self.S_upd = torch.randn(r, r, device="cuda", generator=gen) * 1e-3
        if op in ("step", "apply", "check") and c["reorder"]:
            self.Qx = (torch.empty_like(self.Q[0]), torch.empty_like(self.Q[1]))
            lsp.lsp_projector_reorder(*self.Q, n, d, r, *self.Qx, stream)
        if op in ("step", "compress", "check", "fit", "refresh"):
            self.plan = _bytes(lsp.lsp_plan_bytes(m, n, r, d))
            if op != "refresh":                        # the refresh builds it itself, every time
                lsp.lsp_plan_build(*self.P, *self.Q, m, n, r, d, self.plan, self.plan.numel(), stream)
            self.ws = _bytes(lsp.lsp_compress_planned_workspace_bytes(m, n, r, d))
        if op == "raw":
            self.ws = _bytes(lsp.lsp_compress_workspace_bytes(m, n, r, d))
        if op == "check":
            self.bias_ws = _bytes(lsp.lsp_estimation_bias_workspace_bytes(m, n, r, d))
            self.bias = torch.empty(3, device="cuda")
        if op == "fit":
            self.P_new = (self.P[1] + 0.01 * torch.randn(m, d, device="cuda", generator=gen)).contiguous()
            self.Q_new = (self.Q[1] + 0.01 * torch.randn(n, d, device="cuda", generator=gen)).contiguous()
            self.gP, self.gQ = torch.empty(m, d, device="cuda"), torch.empty(n, d, device="cuda")
            self.fit_ws = _bytes(lsp.lsp_bias_gradient_workspace_bytes(m, n, r, d))
        if op == "refresh":
            self.P_prev = _projector(m, r, d, c["dist"], gen)
            self.Q_prev = _projector(n, r, d, c["dist"], gen)
            self.M_kept = torch.randn(r, r, device="cuda", generator=gen) * 1e-3      # the moments, as the CPU optimiser hands them over
            self.V_kept = torch.rand(r, r, device="cuda", generator=gen) * 1e-6
            self.M, self.V = torch.empty_like(self.M_kept), torch.empty_like(self.V_kept)
            self.status = torch.empty(1, dtype=torch.int32, device="cuda")
            self.build_ws = _bytes(lsp.lsp_plan_build_workspace_bytes(m, n, r, d))
            self.rep_ws = _bytes(lsp.lsp_reproject_state_workspace_bytes(r))


class _State:
    pass


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    st = _State()
    st.op, st.r, st.d, st.code = case["op"], case["r"], case["d"], _CODE[case["dtype"]]
    st.stream = torch.cuda.current_stream()
    st.mats = [_Matrix(case, m, n, gen) for m, n in _shapes(case)]
    st.citems = st.aitems = None
    if len(st.mats) > 1 and st.op in ("step", "compress"):
        st.citems = lsp.compress_items([(x.G, x.plan, x.S, x.ws, x.ws.numel(), x.m, x.n) for x in st.mats])
    if len(st.mats) > 1 and st.op in ("step", "apply"):
        st.aitems = lsp.apply_items([(x.W, x.S_upd, *x.P, *x.Qx, x.m, x.n) for x in st.mats])
    return st


def _compress(st):
    if st.citems is not None:
        lsp.lsp_compress_planned_grouped(st.citems, len(st.mats), st.r, st.d, st.code, st.stream)
    else:
        x = st.mats[0]
        lsp.lsp_compress_planned(x.G, x.plan, x.m, x.n, st.r, st.d, x.S, st.code, x.ws, x.ws.numel(), st.stream)
    return [x.S for x in st.mats]


def _apply(st):
    if st.aitems is not None:
        lsp.lsp_decompress_apply_grouped(st.aitems, len(st.mats), st.r, st.d, st.code, st.stream)
    else:
        x = st.mats[0]
        lsp.lsp_decompress_apply(x.W, x.S_upd, *x.P, *x.Qx, x.m, x.n, st.r, st.d, st.code, st.stream)
    return [x.W for x in st.mats]


def run(st):
    op, x, r, d = st.op, st.mats[0], st.r, st.d
    if op == "step":
        return {"S": _compress(st), "W": _apply(st)}
    if op == "compress":
        return _compress(st)
    if op == "apply":
        return _apply(st)
    if op == "raw":
        lsp.lsp_compress(x.G, *x.P, *x.Q, x.m, x.n, r, d, x.S, st.code, x.ws, x.ws.numel(), st.stream)
        return x.S
    if op == "check":
        S = _compress(st)
        lsp.lsp_estimation_bias(x.G, x.S, *x.P, *x.Qx, x.m, x.n, r, d, x.bias, x.bias_ws, x.bias_ws.numel(), st.code, st.stream)
        return {"S": S, "bias": x.bias}
    if op == "fit":
        lsp.lsp_plan_refresh_values(x.plan, x.P_new, x.Q_new, x.m, x.n, r, d, st.stream)
        lsp.lsp_bias_gradient(x.G, x.plan, x.P[0], x.P_new, x.Q[0], x.Q_new, x.m, x.n, r, d, x.gP, x.gQ,
                              x.fit_ws, x.fit_ws.numel(), st.code, st.stream)
        return {"gP": x.gP, "gQ": x.gQ}
    # refresh: the moments are brought in, the plan of the new projectors is built, the moments follow, and the
    # first gradient goes through the new plan
    x.M.copy_(x.M_kept)
    x.V.copy_(x.V_kept)
    lsp.lsp_plan_build_async(*x.P, *x.Q, x.m, x.n, r, d, x.plan, x.plan.numel(), x.build_ws, x.build_ws.numel(), x.status, st.stream)
    lsp.lsp_reproject_state(*x.P, *x.P_prev, *x.Q, *x.Q_prev, x.m, x.n, r, d, x.M, x.V, x.rep_ws, x.rep_ws.numel(), st.stream)
    return {"status": x.status, "M": x.M, "V": x.V, "S": _compress(st)}


def work(case):
    """Bytes that have to move (each input once, each output once) and operations on the stored entries (Def. 1)."""
    r, d, sz, op = case["r"], case["d"], _SIZE[case["dtype"]], case["op"]
    total = flops = 0.0
    for m, n in _shapes(case):
        ell, mat, sub, half = (m + n) * d * 8, m * n * sz, r * r * 4, 2.0 * m * n * d + 2.0 * m * r * d
        if op in ("step", "compress", "raw", "check", "refresh"):
            total += mat + ell + sub
            flops += half
        if op in ("step", "apply"):
            total += 2 * mat + ell + sub
            flops += half
        if op == "check":
            total += 12
            flops += half + 4.0 * m * n
        if op == "fit":
            total += mat + ell + (m + n) * d * 4
            flops += 4.0 * m * n * d + 2.0 * m * r * d + 10.0 * r ** 3 + 2.0 * (m + n) * d * (d + r)
        if op == "refresh":
            total += ell + 4 * sub
            flops += 8.0 * r ** 3 + 2.0 * (m + n) * d * d
    return {"bytes": total, "flops": flops}


def tolerance(case):
    # S, M, V and the gradients are fp32 sums of up to 1e5 products in another order; W is rounded once to its storage
    # type, so now and then a value falls on the other side of a rounding boundary (one unit in the last place)
    if case["op"] == "fit":
        return {"rel": 5e-5, "max": 2e-3}
    if case["op"] in ("step", "apply") and case["dtype"] == "bf16":
        return {"rel": 2e-3, "max": 1.6e-2}
    if case["op"] in ("step", "apply") and case["dtype"] == "f16":
        return {"rel": 2e-4, "max": 2e-3}
    return {"rel": 1e-5, "max": 4e-4}
