"""2- and 8-bit residual rows in the one-grid kernel, at input widths that take each depth of its own selection and the
selection kernel in front, with last column segments that are not full: against the oracle, like the separate kernels."""
import pytest

import oracle
import workloads
import paper_2412_20185_amd as dd
from helpers import Problem, assert_parity

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rfmt", ["int2", "int8"])
@pytest.mark.parametrize("wfmt,bits,K,N", [("uniform", 3, 4096, 576), ("uniform", 4, 4224, 192), ("lut", 3, 8320, 64),
                                           ("uniform", 3, 16512, 64), ("uniform", 4, 32896, 64)])
def test_one_grid_against_oracle(rfmt, wfmt, bits, K, N):
    p = Problem(workloads.weights(53, 0, 0, K, N), bits, wfmt=wfmt, rfmt=rfmt, lut_iters=2,
                alphas=oracle.quantize.DEFAULT_ALPHAS[::10])
    ws = dd.Workspace(K, N, 4096)
    try:
        for step, k in enumerate([1, 65, 4096]):  # 4096: the largest selection kept in LDS
            x = workloads.x_gauss_outliers(53, 0, 0, step, K)
            y_ref, sc = p.reference(x, k)
            for mode in (dd.MODE_FUSED, dd.MODE_SERIAL):
                ws.set_mode(mode)
                y, idx, _ = p.run(x, k, ws)
                assert_parity(y, y_ref, idx, sc, what=f"{rfmt} {wfmt}{bits} {K}x{N} k={k} mode {mode}")
    finally:
        ws.close()
