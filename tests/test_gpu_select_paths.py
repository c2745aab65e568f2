"""The exact selection on inputs that take each of its ways: by chunks (with and without a list, the list full, one
more than full), with the k-th largest key far above the bound from the chunk maxima, with a bound of zero, and by the
full histograms; stand-alone and inside the one-grid kernel."""
import numpy as np
import pytest
import torch

import oracle
import paper_2412_20185_amd as dd
from paper_2412_20185_amd.layer import StoredLinear

pytestmark = pytest.mark.gpu


def inputs(K):
    """(name, x, ks): chunk = 8 consecutive channels."""
    g = np.random.default_rng(K)
    nchunks = K // 8
    base = (g.standard_normal(K) * 0.05).astype(np.float16)
    yield "gauss", g.standard_normal(K).astype(np.float16), (1, 2, K // 64 + 1, nchunks, min(K, nchunks + 1))
    # one large key in each of `many` chunks: as many listed chunks as there are large keys
    for many in (min(nchunks, 1024), min(nchunks, 1025)):
        x = base.copy()
        at = np.sort(g.choice(nchunks, many, replace=False)) * 8 + g.integers(0, 8, many)
        x[at] = (g.uniform(4, 4.4, many) * g.choice([-1, 1], many)).astype(np.float16)
        yield f"one_in_{many}_chunks", x, (1, many - 1, many, min(nchunks, many + 1))
    # eight large keys in each of a few chunks: the bound from the chunk maxima is far below the k-th largest key
    few = max(1, nchunks // 16)
    x = base.copy()
    for c in g.choice(nchunks, few, replace=False):
        x[8 * c:8 * c + 8] = g.uniform(10, 3000, 8).astype(np.float16)
    yield "crowded", x, (few + 1, min(nchunks, 5 * few), min(nchunks, 8 * few), min(K, 8 * few + 1))
    # keys 255, 256 and 257 above the lower edge of the bound's bin (L = 2.0 = 0x4000)
    x = base.copy()
    x.view(np.uint16)[8 * np.arange(min(nchunks, 40))] = 0x4000
    x.view(np.uint16)[1:1 + 3] = [0x40FE, 0x40FF, 0x4100]
    x.view(np.uint16)[4:7] = [0xC101, 0xC0FF, 0x40FF]
    yield "far_key", x, tuple(range(1, 9))
    # many equal keys, and keys below 2^-17 only (the bound is zero)
    yield "equal", np.full(K, -2.0, np.float16), (1, nchunks // 2 + 1, nchunks)
    t = np.zeros(K, np.float16)
    t.view(np.uint16)[:] = g.integers(0, 128, K)
    yield "tiny", t, (1, nchunks // 3 + 1)


@pytest.mark.parametrize("K", [8, 1000, 2048, 2056, 4096, 4104, 8192, 8200, 16384, 32768, 32776, 65536])
def test_stand_alone(K):
    for name, x, ks in inputs(K):
        xd = torch.from_numpy(x).cuda()
        for k in sorted({k for k in ks if 1 <= k <= K}):
            idx = torch.full((k,), -1, dtype=torch.int32, device="cuda")
            xs = torch.zeros(k, dtype=torch.float16, device="cuda")
            dd.decdec_select_topk(xd, K, k, idx, xs)
            torch.cuda.synchronize()
            sc = oracle.topk_abs(x, k)
            assert np.array_equal(idx.cpu().numpy(), sc), (K, name, k)
            assert np.array_equal(xs.cpu().numpy().view(np.uint16), x[sc].view(np.uint16)), (K, name, k)


@pytest.mark.parametrize("K", [8192, 8200, 16384, 16392, 32768, 32776, 65536])
def test_on_both_sides_of_the_line_between_the_forms(K):
    """k at most a third of the chunks and at most 576 goes by chunks; one more by radix, above 8192 channels in a kernel
    of its own, from which every key of a chunk may be written."""
    x = np.random.default_rng(K + 1).standard_normal(K).astype(np.float16)
    line = min(K // 8 // 3, 576)
    xd = torch.from_numpy(x).cuda()
    for k in (line, line + 1, K - 1, K):
        idx = torch.full((k,), -1, dtype=torch.int32, device="cuda")
        xs = torch.zeros(k, dtype=torch.float16, device="cuda")
        dd.decdec_select_topk(xd, K, k, idx, xs)
        torch.cuda.synchronize()
        sc = oracle.topk_abs(x, k)
        assert np.array_equal(idx.cpu().numpy(), sc), (K, k)
        assert np.array_equal(xs.cpu().numpy().view(np.uint16), x[sc].view(np.uint16)), (K, k)


@pytest.mark.parametrize("K", [128, 4096, 4224, 8192, 8320, 16384, 16512, 32768])
def test_inside_the_one_grid_kernel(K):
    lin = StoredLinear.random(K, 64, 3, dd.W_UNIFORM_G128, 16, seed=1)
    ws = dd.Workspace(K, 64, min(K, 4096))
    y = torch.empty(64, dtype=torch.float16, device="cuda")
    try:
        for name, x, ks in inputs(K):
            xd = torch.from_numpy(x).cuda()
            for k in sorted({k for k in ks if 1 <= k <= min(K, 4096)}):
                lin.gemv(xd, k, y, ws)
                idx, xs = ws.read_selection(k)
                sc = oracle.topk_abs(x, k)
                assert np.array_equal(idx, sc), (K, name, k)
                assert np.array_equal(xs.view(np.uint16), x[sc].view(np.uint16)), (K, name, k)
    finally:
        ws.close()
