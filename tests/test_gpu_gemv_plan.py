"""The base GEMV at sizes that take each branch of its launch plan and leave remainders in it: wavefronts of 16, 32 and 64
columns, groups of input channels that do not fill the last turn, single and many K-slices, and requested turns of more than
one tile.  Against the oracle with the tolerance of all results (fp16 rounding and fp32 sums)."""
import numpy as np
import pytest
import torch

import workloads
import paper_2412_20185_amd as dd
from helpers import Problem, assert_parity

pytestmark = pytest.mark.gpu
NONE = np.zeros(0, np.int32)


@pytest.fixture(autouse=True)
def large_blocks_go_back():
    """Tests elsewhere look at the sizes of device allocations: none of theirs is to be cut from a large one that was freed here."""
    yield
    torch.cuda.empty_cache()


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
    (128, 16384, (256, 256, 1)),     # blocks of 64 columns: one group, three of four wavefronts idle
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


@pytest.mark.parametrize("fmt", ["3", "4", "lut"])
def test_requested_chains_of_turns(fmt):
    """Few wavefronts with many turns keep several tiles on their way: chains of fewer turns than that, one more, multiples
    and remainders of it, and a last wavefront whose chain is shorter than the others' or empty (37 groups)."""
    K, N = 37 * 128, 128
    p = Problem(workloads.weights(58, 0, 0, K, N), 4 if fmt == "4" else 3, wfmt="lut" if fmt == "lut" else "uniform", lut_iters=1)
    x = workloads.x_gauss_outliers(58, 0, 0, 0, K)
    y_ref, _ = p.reference(x, 0)
    ws = dd.Workspace(K, N, 1)
    try:
        for waves, turns in [(w, t) for w in (4, 8, 16) for t in (2, 3, 4, 5, 7, 8, 9, 12, 40)] + [(0, 3), (0, 10), (16, 0)]:
            ws.set_gemv_waves(waves)
            ws.set_gemv_split(turns)
            y, _, _ = p.run(x, 0, ws)
            assert_parity(y, y_ref, NONE, NONE, what=f"{fmt} {waves} x {turns}")
    finally:
        ws.close()


@pytest.mark.parametrize("fmt", ["3", "4", "lut"])
def test_turns_of_the_one_grid_kernel(fmt):
    """Two turns at a time: even and odd chains, and last wavefronts whose chain is cut off."""
    K, N, k = 37 * 128, 128, 40
    p = Problem(workloads.weights(59, 0, 0, K, N), 4 if fmt == "4" else 3, wfmt="lut" if fmt == "lut" else "uniform", lut_iters=1)
    x = workloads.x_gauss_outliers(59, 0, 0, 0, K)
    y_ref, sc = p.reference(x, k)
    ws = dd.Workspace(K, N, k)
    try:
        for turns in (0, 2, 3, 4, 5, 40):
            ws.set_gemv_split(turns)
            y, idx, _ = p.run(x, k, ws)
            assert_parity(y, y_ref, idx, sc, what=f"{fmt} {turns}")
    finally:
        ws.close()


def random_layer(K, N, bits, wfmt):
    """A matrix too large for the oracle, of codes drawn at random, and what it stands for: the fp32 residual of a zero matrix
    is the negative of its weights, decoded by a kernel that shares nothing with the base GEMV."""
    g = torch.Generator(device="cuda").manual_seed(K + N + bits)
    desc = dd.Desc(K, N, bits, wfmt, dd.R_INT4_SYM_COL)
    Wq = torch.randint(0, 256, (dd.decdec_packed_bytes(desc),), dtype=torch.uint8, device="cuda", generator=g)
    lut = wfmt == dd.W_LUT_COL8
    scales = None if lut else (torch.rand((K // 128, N), device="cuda", generator=g) * 0.01 + 0.005).half()
    zl = torch.randn((N, 8) if lut else (K // 128, N), device="cuda", generator=g).mul_(0.02 if lut else 2).half()
    x = torch.randn(K, device="cuda", generator=g).half()
    W_hat = torch.empty((K, N), device="cuda")
    dd.decdec_residual_f32(desc, torch.zeros((K, N), device="cuda"), Wq, scales, zl, W_hat)
    return desc, Wq, scales, zl, x, W_hat.neg_()


def assert_close_to_exact(y, exact, mass):
    """Half a unit in the last place of fp16, and K sums in fp32 of terms that add up to `mass` in absolute value."""
    bound = exact.abs() * 2.0 ** -11 + mass * 2.0 ** -20 + 2.0 ** -24
    assert bool(((y.double() - exact).abs() <= bound).all())


@pytest.mark.parametrize("bits,wfmt", [(3, dd.W_UNIFORM_G128), (4, dd.W_UNIFORM_G128), (3, dd.W_LUT_COL8)])
@pytest.mark.parametrize("K,N,place", [(8192, 24640, "device"), (8320, 24192, "pinned"), (4224, 57344, "pinned")])
def test_one_grid_of_many_rounds(bits, wfmt, K, N, place):
    """Base GEMVs of three rounds of wavefronts, some of whose workgroups take two turns by themselves, the last one cut off."""
    desc, Wq, scales, zl, x, W_hat = random_layer(K, N, bits, wfmt)
    k = 9
    g = torch.Generator(device="cuda").manual_seed(7)
    R = torch.randint(0, 256, (K, N // 2), dtype=torch.uint8, device="cuda", generator=g)
    Rs = (torch.rand(N, device="cuda", generator=g) * 1e-3 + 1e-3).half()
    idx = torch.empty(k, dtype=torch.int32, device="cuda")
    xsel = torch.empty(k, dtype=torch.float16, device="cuda")
    dd.decdec_select_topk(x, K, k, idx, xsel)
    b = R[idx.long()].to(torch.int32)
    q = torch.stack((b & 15, b >> 4), dim=2).view(k, N)
    extra = (q - 16 * (q > 7)).double().mul_(Rs.double()) * xsel.double()[:, None]
    exact = x.double() @ W_hat.double() + extra.sum(0)
    mass = x.double().abs() @ W_hat.double().abs() + extra.abs().sum(0)
    # the weights are differences of code and zero point, of which the kernel adds up the terms apart
    if scales is not None:
        mass += (scales.double() * (2 ** bits + zl.double().abs())).repeat_interleave(128, 0).mul_(x.double().abs()[:, None]).sum(0)
    if place == "pinned":
        host = torch.empty(R.shape, dtype=R.dtype, pin_memory=True)
        R = host.copy_(R)
    ws = dd.Workspace(K, N, k)
    try:
        for _ in range(2):
            y = torch.full((N,), float("nan"), dtype=torch.float16, device="cuda")
            dd.decdec_gemv(desc, x, Wq, scales, zl, R, Rs, k, y, ws)
            assert_close_to_exact(y, exact, mass)
    finally:
        ws.close()


@pytest.mark.parametrize("K,N,launches", [  # workgroups, threads, columns, K-slices; the same or in 3 bits, 4 bits, with codebooks
    (1152, 16384, [(256, 1024, 64, 1)]),   # nine groups by nine of 16 wavefronts
    (2176, 32768, [(512, 1024, 64, 1)]),   # 17 groups by nine wavefronts, the last with one
    (4096, 28672, [(448, 1024, 64, 1)]),   # two groups by each of 16
    (3968, 28672, [(448, 1024, 64, 1)]),   # 31 groups: the last wavefront with one
    (2560, 40960, [(2560, 512, 16, 1)]),   # 2.5 rounds of 64 columns: blocks of 16
    (1408, 47168, [(737, 512, 64, 1)]),    # 11 groups, two by each of six wavefronts
    (256, 43072, [(673, 256, 64, 1)]),     # two groups: always blocks of 64, two of four wavefronts idle
    (1024, 18176, [(1136, 256, 16, 1)]),   # just above one round: blocks of 16
    (8320, 28288, [(3978, 512, 64, 9), (3978, 512, 64, 9), (2210, 512, 64, 5)]),        # codebooks: slices of two turns
    (16640, 6208, [(1746, 512, 32, 9), (1746, 512, 32, 9), (873, 512, 64, 9)]),
    (16640, 24256, [(3411, 512, 64, 9), (6822, 512, 32, 9), (3411, 512, 64, 9)]),       # in 3 bits too
])
@pytest.mark.parametrize("bits,wfmt", [(3, dd.W_UNIFORM_G128), (4, dd.W_UNIFORM_G128), (3, dd.W_LUT_COL8)])
def test_wide_matrices(bits, wfmt, K, N, launches):
    """Matrices too large for the oracle: the plan's choice and K-slices added by atomics against sums in fp64."""
    desc, Wq, scales, zl, x, W_hat = random_layer(K, N, bits, wfmt)
    exact, mass = x.double() @ W_hat.double(), x.double().abs() @ W_hat.double().abs()
    # the weights are differences of code and zero point, of which the kernel adds up the terms apart
    if scales is not None:
        mass += (scales.double() * (2 ** bits + zl.double().abs())).repeat_interleave(128, 0).mul_(x.double().abs()[:, None]).sum(0)
    ws = dd.Workspace(K, N, 1)
    try:
        launch = launches[-1 if wfmt == dd.W_LUT_COL8 else (bits - 3) % len(launches)]
        assert ws.gemv_launch_shape_of(desc) == launch
        assert (bits, wfmt) != (3, dd.W_UNIFORM_G128) or ws.gemv_launch_shape(K, N) == launch[:2] + (64 // launch[2] * launch[3],)
        for waves in (0, 4):
            ws.set_gemv_waves(waves)
            y = torch.full((N,), float("nan"), dtype=torch.float16, device="cuda")
            dd.decdec_gemv(desc, x, Wq, scales, zl, None, None, 0, y, ws)
            assert_close_to_exact(y, exact, mass)
    finally:
        ws.close()
