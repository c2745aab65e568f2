"""The work that a program built on this library has it do, as cases that can be timed and compared.

Four kinds, each through the public calls:

  step     the linear layers of a decode step at batch 1: per layer q+k+v, o, gate+up and down, as four
           decdec_gemv_multi calls, captured once into a HIP graph and replayed per token (how a decoder runs
           them), or issued eagerly.  Residual rows in pinned host memory (the method's placement), in GPU
           memory (the option for a GPU with room), or no compensation at all.
  linear   one linear layer, eagerly: decdec_gemv, the allocation-free decdec_gemv_static, or a selection made
           once (exact or bucket) and handed to decdec_gemv_idx.
  select   the exact top-k alone.
  prepare  a layer made ready from its fp32 weights: quantiser, residual, residual quantiser (UniformLinear).

Sizes are those of the layer shapes and settings in `workloads` and `bench.py`, and generic ones between them.
"""
from __future__ import annotations

import math

import torch

import paper_2412_20185_amd as dd
from paper_2412_20185_amd.layer import LinearGroup, StoredLinear, UniformLinear

W_SIGMA = 0.02          # weights are N(0, 0.02^2)
LAYER_8B = dict(hidden=4096, kv=1024, inter=14336)
LAYER_70B = dict(hidden=8192, kv=1024, inter=28672)


def listed():
    return [
        # The smallest call: one 1024 x 1024 layer, 4-bit weights, fp16 residual rows, k = 32.  Launch latency.
        dict(name="linear_1024", kind="linear", entry="gemv", K=1024, N=1024, wbits=4, lut=False, rbits=16, k=32,
             place="pinned"),
        # A serving loop that must not allocate: one 4096 x 4096 layer with the method's own 4-bit residual rows.
        dict(name="linear_static_4096", kind="linear", entry="static", K=4096, N=4096, wbits=3, lut=False, rbits=4,
             k=60, place="pinned"),
        # A ragged layer: 25 groups of input channels, 135 tiles of output columns, a last column segment that is
        # not full, selection made by a call of its own.
        dict(name="linear_idx_ragged", kind="linear", entry="idx", K=3200, N=8640, wbits=4, lut=False, rbits=4, k=50,
             place="pinned"),
        # A down projection with 8-bit residual rows (the bit-width study).
        dict(name="linear_down_int8", kind="linear", entry="gemv", K=14336, N=4096, wbits=3, lut=False, rbits=8, k=56,
             place="pinned"),
        # The exact top-k alone at the widest input of the 70B-sized layer.
        dict(name="select_28672", kind="select", K=28672, k=286),
        # 32 layers without compensation: what the base GEMVs cost per token.
        dict(name="step_8b_base", kind="step", layers=32, wbits=3, lut=False, rbits=16, k_per_1024=0.0,
             place="none", graph=True, **LAYER_8B),
        # The benchmark's step: fp16 rows over the host link, k = 2 % of the channels.
        dict(name="step_8b_fp16_2pct", kind="step", layers=2, wbits=3, lut=False, rbits=16, k_per_1024=20.48,
             place="pinned", graph=True, **LAYER_8B),
        # The method's residual format near the point where compensation is cheap (2 % of the weight bytes).
        dict(name="step_8b_int4_15", kind="step", layers=8, wbits=3, lut=False, rbits=4, k_per_1024=15.0,
             place="pinned", graph=True, **LAYER_8B),
        # Residual rows kept in GPU memory, 4-bit weights.
        dict(name="step_8b_hbm", kind="step", layers=4, wbits=4, lut=False, rbits=16, k_per_1024=20.48,
             place="device", graph=True, **LAYER_8B),
        # The largest layer: 70B-sized, codebook weights, fp16 rows, k = 1 %.
        dict(name="step_70b_lut", kind="step", layers=1, wbits=3, lut=True, rbits=16, k_per_1024=10.24,
             place="pinned", graph=True, **LAYER_70B),
        # A model being made ready: one square layer with the residual quantiser, ...
        dict(name="prepare_int4", kind="prepare", K=4096, N=4096, wbits=3, rbits=4),
        # ... and one wide layer with fp16 residual rows.
        dict(name="prepare_fp16", kind="prepare", K=4096, N=14336, wbits=4, rbits=16),
    ]


def _log_int(rng, lo, hi, multiple):
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return min(hi, max(lo, int(round(v / multiple)) * multiple))


def draw(rng):
    kind = rng.choice(("step", "step", "linear", "linear", "linear", "select", "prepare"))
    lut = rng.random() < 0.3
    wbits = 3 if lut else rng.choice((3, 4))
    if kind == "select":
        K = _log_int(rng, 1024, 32768, 8)
        return dict(kind=kind, K=K, k=_log_int(rng, 1, max(1, K // 16), 1))
    if kind == "prepare":
        return dict(kind=kind, K=_log_int(rng, 256, 4096, 128), N=_log_int(rng, 256, 4096, 64), wbits=rng.choice((3, 4)),
                    rbits=rng.choice((2, 4, 4, 8, 16)))
    if kind == "linear":
        entry = rng.choice(("gemv", "gemv", "static", "idx", "bucket"))
        K = _log_int(rng, 1024, 28672, 1024 if entry == "bucket" else 128)
        N = _log_int(rng, 256, 16384, 64)
        k = (K // 1024) * rng.randint(1, 24) if entry == "bucket" else _log_int(rng, 1, max(1, K // 32), 1)
        return dict(kind=kind, entry=entry, K=K, N=N, wbits=wbits, lut=lut, rbits=rng.choice((16, 4, 4, 2, 8)), k=k,
                    place=rng.choice(("pinned", "pinned", "device")))
    hidden = _log_int(rng, 1024, 6144, 128)
    inter = int(round(hidden * rng.uniform(2.5, 3.6) / 128)) * 128
    kv = max(64, int(round(hidden / rng.choice((1, 4, 8)) / 64)) * 64)
    place = rng.choice(("pinned", "pinned", "device", "none"))
    return dict(kind="step", layers=rng.randint(1, 4), hidden=hidden, kv=kv, inter=inter, wbits=wbits, lut=lut,
                rbits=rng.choice((16, 4, 4)), k_per_1024=0.0 if place == "none" else round(math.exp(rng.uniform(0, math.log(24))), 2),
                place=place, graph=rng.random() < 0.8)


# ------------------------------------------------------------------ inputs

def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _activations(g, *shape):
    """fp16 ~ N(0, 1) with 0.5 % of the channels 10 to 50 times as large, at positions of their own in every vector."""
    x = torch.randn(shape, device="cuda", generator=g)
    gain = torch.rand(shape, device="cuda", generator=g) * 40 + 10
    return torch.where(torch.rand(shape, device="cuda", generator=g) < 0.005, x * gain, x).half()


def _residual_rows(R, rbits):
    """The rows of R in the library's residual formats, on the GPU: fp16, or packed symmetric codes and their column scales."""
    if rbits == 16:
        return R.half(), None
    qmax = 2 ** (rbits - 1) - 1
    scale = (R.abs().amax(0) * (0.85 / qmax)).clamp_min(1e-6).half()
    q = (R / scale.float()).round_().clamp_(-qmax, qmax).to(torch.int8)
    if rbits < 8:
        per = 8 // rbits
        q = q.view(R.shape[0], -1, per) & (2 ** rbits - 1)
        byte = q[..., 0].clone()
        for i in range(1, per):
            byte |= q[..., i] << (rbits * i)
        q = byte
    return q.view(torch.uint8), scale


def _linear(g, K, N, wbits, lut, rbits, place):
    """A stored layer: weights drawn and quantised on the GPU (codebook weights: random codes and an ascending codebook per column)."""
    wfmt = dd.W_LUT_COL8 if lut else dd.W_UNIFORM_G128
    desc = dd.Desc(K, N, wbits, wfmt, dd.R_FMT_OF_BITS[rbits])
    Wq = torch.empty(dd.decdec_packed_bytes(desc), dtype=torch.uint8, device="cuda")
    R = scales = None
    if lut:
        Wq.random_(0, 256, generator=g)
        zl = (torch.sort(torch.randn((N, 8), device="cuda", generator=g), dim=1).values * W_SIGMA).half()
        if place != "none":
            R = torch.randn((K, N), device="cuda", generator=g) * (W_SIGMA * 0.15)
    else:
        W = torch.randn((K, N), device="cuda", generator=g) * W_SIGMA
        scales = torch.empty((K // 128, N), dtype=torch.float16, device="cuda")
        zl = torch.empty((K // 128, N), dtype=torch.float16, device="cuda")
        dd.decdec_quantize_uniform(desc, W, Wq, scales, zl, None)
        if place != "none":
            R = torch.empty((K, N), device="cuda")
            dd.decdec_residual_f32(desc, W, Wq, scales, zl, R)
    rows = row_scales = None
    if place != "none":
        rows, row_scales = _residual_rows(R, rbits)
        if place == "pinned":
            host = torch.empty(rows.shape, dtype=rows.dtype, pin_memory=True)
            host.copy_(rows)
            rows = host
    return StoredLinear(desc, Wq, scales, zl, rows, row_scales, rbits)


def _calls(case):
    """(input channels, output channels of each matrix) of the four calls of a layer."""
    h, kv, f = case["hidden"], case["kv"], case["inter"]
    return [(h, [h, kv, kv]), (h, [h]), (h, [f, f]), (f, [h])]


def _k_of(case, K):
    return 0 if case["place"] == "none" else max(1, int(K * case["k_per_1024"] / 1024 + 1e-9))


def prepare(case, seed):
    g = _generator(seed)
    st = dict(case=case)
    if case["kind"] == "select":
        st["x"] = _activations(g, case["K"])
        st["idx"] = torch.empty(case["k"], dtype=torch.int32, device="cuda")
        st["xsel"] = torch.empty(case["k"], dtype=torch.float16, device="cuda")
        return st
    if case["kind"] == "prepare":
        st["W"] = torch.randn((case["K"], case["N"]), device="cuda", generator=g) * W_SIGMA
        return st
    if case["kind"] == "linear":
        K, N, k = case["K"], case["N"], case["k"]
        st["lin"] = _linear(g, K, N, case["wbits"], case["lut"], case["rbits"], case["place"])
        st["x"] = _activations(g, K)
        st["y"] = torch.empty(N, dtype=torch.float16, device="cuda")
        if case["entry"] != "static":
            st["ws"] = dd.Workspace(K, N, k)
        if case["entry"] in ("idx", "bucket"):
            st["idx"] = torch.empty(k, dtype=torch.int32, device="cuda")
            st["xsel"] = torch.empty(k, dtype=torch.float16, device="cuda")
        if case["entry"] == "bucket":  # the two boundaries, calibrated on other activations of the same kind
            a = torch.sort(_activations(g, 8, K).float().abs(), dim=1, descending=True).values
            st["b0"], st["b15"] = float(a[:, 0].max()), float(a[:, k - 1].max())
        torch.cuda.synchronize()
        return st

    calls, L = _calls(case), case["layers"]
    st["x"] = [_activations(g, L, K) for K, _ in calls]
    st["y"] = torch.empty((L, sum(sum(Ns) for _, Ns in calls)), dtype=torch.float16, device="cuda")
    st["ws"] = dd.Workspace(max(K for K, _ in calls), max(sum(Ns) for _, Ns in calls), max(_k_of(case, K) for K, _ in calls))
    st["groups"] = []
    for layer in range(L):
        at = 0
        for c, (K, Ns) in enumerate(calls):
            lins, ys = [], []
            for N in Ns:
                lins.append(_linear(g, K, N, case["wbits"], case["lut"], case["rbits"], case["place"]))
                ys.append(st["y"][layer, at:at + N])
                at += N
            st["groups"].append((LinearGroup(lins, ys), st["x"][c][layer], _k_of(case, K)))
    torch.cuda.synchronize()
    if case["graph"]:
        st["graph"] = torch.cuda.CUDAGraph()
        with torch.cuda.graph(st["graph"]):
            _step(st)
    return st


# ------------------------------------------------------------------ one pass

def _step(st):
    for group, x, k in st["groups"]:
        group.gemv(x, k, st["ws"])


def run(st):
    case = st["case"]
    if case["kind"] == "step":
        if case["graph"]:
            st["graph"].replay()
        else:
            _step(st)
        return st["y"]
    if case["kind"] == "select":
        dd.decdec_select_topk(st["x"], case["K"], case["k"], st["idx"], st["xsel"])
        return st["idx"], st["xsel"]
    if case["kind"] == "prepare":
        lin = UniformLinear(st["W"], case["wbits"], rbits=case["rbits"])
        return lin.Wq, lin.scales, lin.zeros, lin.R, lin.R_scales
    lin, x, y, k = st["lin"], st["x"], st["y"], case["k"]
    if case["entry"] == "gemv":
        lin.gemv(x, k, y, st["ws"])
        return y
    if case["entry"] == "static":
        dd.decdec_gemv_static(lin.desc, x, lin.Wq, lin.scales, lin.zeros, lin.R, lin.R_scales, k, y)
        return y
    if case["entry"] == "idx":
        dd.decdec_select_topk(x, case["K"], k, st["idx"], st["xsel"])
    else:
        dd.decdec_select_bucket(x, case["K"], k // (case["K"] // 1024), st["b0"], st["b15"], st["idx"], st["xsel"])
    dd.decdec_gemv_idx(lin.desc, x, lin.Wq, lin.scales, lin.zeros, lin.R, lin.R_scales, k, st["idx"], st["xsel"], y,
                       st["ws"])
    return y, st["idx"], st["xsel"]


# ------------------------------------------------------------------ what a pass is worth

def _gemv_work(case, K, Ns, k):
    """Packed codes, scales and zero points (or codebooks), x and y; the selected rows and their column scales."""
    N = sum(Ns)
    meta = 16 * N if case["lut"] else 4 * N * (K // 128)
    rows = k * N * case["rbits"] // 8 + (2 * N if k and case["rbits"] != 16 else 0)
    return K * N * case["wbits"] // 8 + meta + 2 * K + 2 * N + rows, 2 * K * N + 2 * k * N


def work(case):
    if case["kind"] == "select":
        return dict(bytes=2 * case["K"] + 6 * case["k"], flops=0)
    if case["kind"] == "prepare":
        K, N, r = case["K"], case["N"], case["rbits"]
        by = 4 * K * N + K * N * case["wbits"] // 8 + 4 * N * (K // 128) + K * N * r // 8 + (0 if r == 16 else 2 * N)
        # per weight: two for the range, four for code and residual; the scale search: 71 scales, seven each
        return dict(bytes=by, flops=K * N * (6 + (0 if r == 16 else 71 * 7)))
    if case["kind"] == "linear":
        by, fl = _gemv_work(case, case["K"], [case["N"]], case["k"])
        return dict(bytes=by + (6 * case["k"] if case["entry"] in ("idx", "bucket") else 0), flops=fl)
    parts = [_gemv_work(case, K, Ns, _k_of(case, K)) for K, Ns in _calls(case)]
    return dict(bytes=case["layers"] * sum(p[0] for p in parts), flops=case["layers"] * sum(p[1] for p in parts))


def tolerance(case):
    # Selections, codes and scales are defined bit for bit.
    if case["kind"] in ("select", "prepare"):
        return "exact"
    # y is fp16: against the same sums in fp64 the two-norm is off by 2.1e-4 and the worst value by half a unit in the last
    # place, 4.9e-4 of it.
    return {"rel": 8e-4, "max": 2e-3}
