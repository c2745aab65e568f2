"""The base GEMV at sizes that take each branch of its launch plan and leave remainders in it: wavefronts of 16, 32 and 64
columns, groups of input channels that do not fill the last turn, single and many K-slices, and requested turns of more than
one tile.  Against the oracle with the tolerance of all results (fp16 rounding and fp32 sums)."""
import numpy as np
import pytest

import workloads
import paper_2412_20185_amd as dd
from helpers import Problem, assert_parity

pytestmark = pytest.mark.gpu
NONE = np.zeros(0, np.int32)


@pytest.mark.parametrize("fmt", ["3", "4", "lut"])
@pytest.mark.parametrize("K,N,launch", [
    (128, 64, (4, 256, 4)),           # one group: blocks of 16 columns, one wavefront
    (640, 2112, (132, 256, 4)),      # five groups by two wavefronts of four; 132 blocks, the last four in their own order
    (384, 4160, (130, 256, 2)),      # 260 blocks of 16 columns would take two rounds: blocks of 32, the last group alone
    (4352, 2048, (128, 1024, 4)),     # nine wavefronts over all of K
    (4480, 64, (9, 256, 9)),         # K-slices of four wavefronts, the last with three groups
    (8320, 64, (13, 512, 13)),       # 65 groups: up to 16 slices
    (16512, 64, (18, 512, 18)),      # 129 groups: blocks of 32 columns, nine slices
    (33024, 64, (36, 512, 36)),      # 258 groups: blocks of 16 columns, nine slices
])
def test_base_gemv_against_oracle(fmt, K, N, launch):
    p = Problem(workloads.weights(57, 0, 0, K, N), 4 if fmt == "4" else 3, wfmt="lut" if fmt == "lut" else "uniform", lut_iters=1)
    ws = dd.Workspace(K, N, 1)
    try:
        assert ws.gemv_launch_shape(K, N) == launch
        for step in range(2):
            x = workloads.x_gauss_outliers(57, 0, 0, step, K)
            y, _, _ = p.run(x, 0, ws)
            y_ref, _ = p.reference(x, 0)
            assert_parity(y, y_ref, NONE, NONE, what=f"{fmt} {K}x{N}")
            for waves, turns in ((4, 3), (16, 2), (8, 1)):
                ws.set_gemv_waves(waves)
                ws.set_gemv_split(turns)
                y, _, _ = p.run(x, 0, ws)
                assert_parity(y, y_ref, NONE, NONE, what=f"{fmt} {K}x{N} {waves} x {turns}")
            ws.set_gemv_waves(0)
            ws.set_gemv_split(0)
    finally:
        ws.close()
