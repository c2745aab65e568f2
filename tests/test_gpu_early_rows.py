"""Rows that are requested before the selection is complete: selections of which all, some and none of the requested rows are
part, ties at the cut, shares of several workgroups, against the oracle and bit for bit against rows requested after it."""
import numpy as np
import pytest
import torch

import oracle
import workloads
import paper_2412_20185_amd as dd
from helpers import RFMT, Problem, assert_parity, fetch_plan
from paper_2412_20185_amd.layer import StoredLinear

pytestmark = pytest.mark.gpu


def activations(K, k):
    """(name, x)"""
    g = np.random.default_rng(K + k)
    yield "outliers", workloads.x_gauss_outliers(71, 0, 0, 0, K)
    # the k largest crowd in k / 4 chunks of 8, so that many chunks whose maximum is among the k largest maxima hold no
    # selected channel
    x = g.uniform(1.0, 3.9, K).astype(np.float16)
    for c in g.choice(K // 8, max(1, k // 4), replace=False):
        x[8 * c:8 * c + 4] = g.uniform(4, 60, 4).astype(np.float16)
    yield "crowded", x
    # all in one wavefront's run of channels, and in the last one
    for name, at in (("first", 0), ("last", K - 4 * k)):
        x = (g.standard_normal(K) * 0.05).astype(np.float16)
        x[at:at + 4 * k] += (g.uniform(1, 40, 4 * k) * (g.random(4 * k) < 0.4)).astype(np.float16)
        yield name, x
    # few distinct magnitudes: ties at the cut, also among the requested
    x = g.choice([0.5, 1.0, 2.0, 8.0], K, p=[0.9, 0.06, 0.03, 0.01]).astype(np.float16) * g.choice([-1, 1], K).astype(np.float16)
    yield "ties", x
    yield "zero", np.zeros(K, np.float16)
    yield "equal", np.full(K, -1.5, np.float16)


@pytest.mark.parametrize("rfmt,K,N,k", [("fp16", 4096, 1600, 81), ("int8", 4096, 2112, 60), ("int4", 4096, 4160, 61),
                                        ("int4", 8320, 2048, 100), ("int8", 16384, 2112, 200), ("fp16", 2048, 4096, 85),
                                        ("int4", 1024, 28672, 5),
                                        # two and four chunks of keys per thread; fp16 rows whose sums are added after a look
                                        ("fp16", 4096, 5696, 90), ("fp16", 4224, 5184, 90), ("fp16", 6144, 3648, 90), ("int8", 6144, 4160, 90), ("int4", 6144, 2048, 90),
                                        ("fp16", 8320, 3648, 140), ("int8", 8320, 4160, 100)])
def test_early_rows(rfmt, K, N, k):
    assert fetch_plan(RFMT[rfmt], K, [N], k).early > 0
    g = np.random.default_rng(N)
    W = workloads.weights(71, 0, 0, K, N) if K * N < 1 << 23 else (g.standard_normal((K, N), dtype=np.float32) * 0.02)
    p = Problem(W, 4, rfmt=rfmt, alphas=oracle.quantize.DEFAULT_ALPHAS[::35])
    ws = dd.Workspace(K, N, k)
    try:
        for name, x in activations(K, k):
            y_ref, sc = p.reference(x, k)
            ws.set_separate_select(True)
            y_a, idx_a, _ = p.run(x, k, ws)
            ws.set_separate_select(False)
            for mode in (dd.MODE_FUSED, dd.MODE_SERIAL):
                ws.set_mode(mode)
                y, idx, xs = p.run(x, k, ws)
                assert np.array_equal(xs.view(np.uint16), x[sc].view(np.uint16)), name
                if name != "zero":
                    assert_parity(y, y_ref, idx, sc, what=f"{name} mode {mode}")
                else:
                    assert np.array_equal(idx, sc) and not y.any()
                if mode == dd.MODE_FUSED:
                    assert np.array_equal(y.view(np.uint16), y_a.view(np.uint16)), name
            ws.set_mode(dd.MODE_FUSED)
    finally:
        ws.close()


def test_infinite_activations():
    """An infinite and a NaN activation are selected first; the columns hold what the products give, as without early rows."""
    K, N, k = 4096, 4096, 60
    assert fetch_plan(dd.R_FP16, K, [N], k).early > 0
    p = Problem(workloads.weights(72, 0, 0, K, N), 4)
    x = workloads.x_gauss_outliers(72, 0, 0, 0, K)
    x[[7, 2000]] = [np.inf, -np.inf]
    x[3100] = np.nan
    ws = dd.Workspace(K, N, k)
    try:
        ws.set_separate_select(True)
        y_a, idx_a, _ = p.run(x, k, ws)
        ws.set_separate_select(False)
        y_b, idx_b, _ = p.run(x, k, ws)
        assert np.array_equal(idx_a, idx_b) and {7, 2000, 3100} <= set(idx_b.tolist())
        assert np.array_equal(y_a.view(np.uint16), y_b.view(np.uint16))
    finally:
        ws.close()


@pytest.mark.parametrize("rbits,K,N,k", [(16, 2048, 9728, 85), (16, 4096, 13824, 81), (16, 4096, 16384, 60), (8, 4096, 9728, 60),
                                         (8, 4096, 20992, 64), (8, 4096, 20992, 65), (8, 2048, 28672, 85), (4, 4096, 10240, 60),
                                         (4, 2048, 28672, 80)])
def test_same_bits_whoever_selects(rbits, K, N, k):
    """17 to 56 segments, where a workgroup has three to seven wavefronts for the rows, or all eight."""
    lin = StoredLinear.random(K, N, 3, dd.W_UNIFORM_G128, rbits, seed=3)
    ws = dd.Workspace(K, N, k)
    y = [torch.full((N,), float("nan"), dtype=torch.float16, device="cuda") for _ in range(3)]
    try:
        for seed in range(4):
            x = torch.from_numpy(workloads.x_gauss_outliers(73, seed, 0, 0, K)).cuda()
            lin.gemv(x, k, y[0], ws)
            ws.set_separate_select(True)
            lin.gemv(x, k, y[1], ws)
            ws.set_separate_select(False)
            idx, xsel = (torch.from_numpy(a).cuda() for a in ws.read_selection(k))
            dd.decdec_gemv_idx(lin.desc, x, lin.Wq, lin.scales, lin.zeros, lin.R, lin.R_scales, k, idx, xsel, y[2], ws)
            for other in y[1:]:
                assert torch.equal(y[0].view(torch.int16), other.view(torch.int16)), seed
    finally:
        ws.close()
