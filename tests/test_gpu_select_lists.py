"""The selection's lists of chunks, one per wavefront: all that may be selected in the run of one wavefront, as many as its list
holds, as it holds when it is filled twice, and one more of each, up to the whole run; stand-alone and inside the one-grid kernel.
And channels ordered by magnitude, where the first wavefronts have most of them."""
import numpy as np
import pytest
import torch

import oracle
import paper_2412_20185_amd as dd
from paper_2412_20185_amd.layer import StoredLinear

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K,run,held", [(8192, 128, 128), (16384, 256, 128), (28672, 512, 192), (32768, 512, 192), (40960, 512, 128),
                                        (16512, 258, 192)])  # the last: runs of the stand-alone kernel from k = 201 on
def test_list_of_one_wavefront(K, run, held):
    """run: chunks of a wavefront; held: entries of its list."""
    g = np.random.default_rng(K)
    lin = StoredLinear.random(K, 64, 3, dd.W_UNIFORM_G128, 16, seed=1) if K <= 32768 else None
    ws = dd.Workspace(K, 64, 576)
    y = torch.empty(64, dtype=torch.float16, device="cuda")
    try:
        for wave in (0, K // 8 // run - 1):  # the first, and the last with a whole run
            for many in (held - 1, held, held + 1, held + 65, 2 * held, 2 * held + 1, run):
                x = (g.standard_normal(K) * 0.05).astype(np.float16)
                at = (wave * run + np.sort(g.choice(run, min(many, run), replace=False))) * 8 + g.integers(0, 8, min(many, run))
                x[at] = (g.uniform(4, 4.4, at.size) * g.choice([-1, 1], at.size)).astype(np.float16)
                xd = torch.from_numpy(x).cuda()
                for k in sorted({1, min(at.size, 200), min(at.size, 500, K // 24)}):
                    sc = oracle.topk_abs(x, k)
                    idx = torch.full((k,), -1, dtype=torch.int32, device="cuda")
                    xs = torch.zeros(k, dtype=torch.float16, device="cuda")
                    dd.decdec_select_topk(xd, K, k, idx, xs)
                    torch.cuda.synchronize()
                    assert np.array_equal(idx.cpu().numpy(), sc), (wave, many, k)
                    assert np.array_equal(xs.cpu().numpy().view(np.uint16), x[sc].view(np.uint16)), (wave, many, k)
                    if lin is not None:
                        lin.gemv(xd, k, y, ws)
                        idx, xs = ws.read_selection(k)
                        assert np.array_equal(idx, sc), (wave, many, k)
                        assert np.array_equal(xs.view(np.uint16), x[sc].view(np.uint16)), (wave, many, k)
    finally:
        ws.close()


@pytest.mark.parametrize("K,ks", [(8192, (81, 341)), (14336, (143, 210, 286, 576)), (20480, (200, 201, 576)), (28672, (286, 576))])
def test_channels_ordered_by_magnitude(K, ks):
    lin = StoredLinear.random(K, 64, 3, dd.W_UNIFORM_G128, 16, seed=1)
    ws = dd.Workspace(K, 64, 576)
    y = torch.empty(64, dtype=torch.float16, device="cuda")
    g = np.random.default_rng(K)
    try:
        for fall in (-2.0, 1.0, 2.0, 4.0):
            x = (g.standard_normal(K) * np.exp(-fall * np.arange(K) / K)).astype(np.float16)
            xd = torch.from_numpy(x).cuda()
            for k in ks:
                sc = oracle.topk_abs(x, k)
                idx = torch.full((k,), -1, dtype=torch.int32, device="cuda")
                xs = torch.zeros(k, dtype=torch.float16, device="cuda")
                dd.decdec_select_topk(xd, K, k, idx, xs)
                lin.gemv(xd, k, y, ws)
                for i, v in ((idx.cpu().numpy(), xs.cpu().numpy()), ws.read_selection(k)):
                    assert np.array_equal(i, sc), (fall, k)
                    assert np.array_equal(v.view(np.uint16), x[sc].view(np.uint16)), (fall, k)
    finally:
        ws.close()
