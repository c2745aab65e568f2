"""GPU parity of the device quantiser: codes, scales, zero points and the fp16
residual must equal the oracle's bit for bit (every decision is one IEEE fp32
operation on both sides)."""
import numpy as np
import pytest
import torch

import oracle
import workloads
import paper_2412_20185_amd as dd
from paper_2412_20185_amd.layer import UniformLinear

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bits", [3, 4])
@pytest.mark.parametrize("K,N", [(1024, 1024), (384, 192), (4096, 1024)])
def test_quantiser_matches_oracle_bit_for_bit(bits, K, N):
    W = workloads.weights(70 + bits, 0, 0, K, N)
    W[128:256, 3] = 0.0125          # constant group: scale 0 -> 1
    W[0:128, 5] *= 1e-4             # tiny range: subnormal fp16 scale
    lin = UniformLinear(W, bits)
    codes, s, z = oracle.quantize_uniform(W, bits)
    assert np.array_equal(lin.scales.cpu().numpy().view(np.uint16), s.view(np.uint16))
    assert np.array_equal(lin.zeros.cpu().numpy().view(np.uint16), z.view(np.uint16))
    packed = lin.Wq.cpu().numpy()
    assert np.array_equal(dd.decdec_unpack_weights(lin.desc, packed), codes)
    assert np.array_equal(packed, dd.decdec_pack_weights(lin.desc, codes))
    R = oracle.residual_fp16(W, oracle.dequantize_uniform(codes, s, z))
    assert np.array_equal(lin.R.numpy().view(np.uint16), R.view(np.uint16))


def _residual_f32_reference(W, W_hat):
    """fp32 of W - W_hat (the difference itself is exact in fp64 for these magnitudes)."""
    return (W.astype(np.float64) - W_hat).astype(np.float32)


@pytest.mark.parametrize("wfmt,bits", [("uniform", 3), ("uniform", 4), ("lut", 3)])
def test_residual_f32_of_packed_weights(wfmt, bits):
    """R = W - W_hat from the packed weights, whatever base quantiser produced them."""
    K, N = 640, 192
    W = workloads.weights(75, 0, 0, K, N)
    if wfmt == "uniform":
        codes, s, z = oracle.quantize_uniform(W, bits)
        W_hat = oracle.dequantize_uniform(codes, s, z)
        desc = dd.Desc(K, N, bits)
        s_d, zl_d = torch.from_numpy(s).cuda(), torch.from_numpy(z).cuda()
    else:
        codes, lut = oracle.quantize_lut(W, iters=2)
        W_hat = oracle.dequantize_lut(codes, lut)
        desc = dd.Desc(K, N, 3, dd.W_LUT_COL8)
        s_d, zl_d = None, torch.from_numpy(lut).cuda()
    Wq = torch.from_numpy(dd.decdec_pack_weights(desc, codes)).cuda()
    R = torch.full((K, N), float("nan"), dtype=torch.float32, device="cuda")
    dd.decdec_residual_f32(desc, torch.from_numpy(W).cuda(), Wq, s_d, zl_d, R)
    torch.cuda.synchronize()
    assert np.array_equal(R.cpu().numpy().view(np.uint32), _residual_f32_reference(W, W_hat).view(np.uint32))


@pytest.mark.parametrize("rbits", [2, 4, 8])
@pytest.mark.parametrize("K,N", [(1024, 512), (384, 192)])
def test_residual_quantiser_matches_oracle_bit_for_bit(rbits, K, N):
    """Section 4.2's quantiser and its 2- and 8-bit variants: scales and codes equal the oracle's.
    Both sides decide in fp64, one IEEE operation per step, column errors summed in ascending k."""
    g = np.random.default_rng([76, rbits, K])
    R32 = (g.standard_normal((K, N)) * 2e-3).astype(np.float32)
    R32[:, 3] = 0.0                       # all-zero column: S = 1
    R32[:, 5] *= 1e-5                     # subnormal fp16 scales
    R32[7, 9] = 0.05                      # one outlier: the search clips it
    q_ref, S_ref = oracle.quantize_residual_sym(R32.astype(np.float64), rbits)
    codes = torch.zeros((K, N * rbits // 8), dtype=torch.uint8, pin_memory=True)
    S = torch.zeros(N, dtype=torch.float16, device="cuda")
    dd.decdec_quantize_residual(K, N, rbits, torch.from_numpy(R32).cuda(), codes, S)
    torch.cuda.synchronize()
    assert np.array_equal(S.cpu().numpy().view(np.uint16), S_ref.view(np.uint16))
    assert np.array_equal(codes.numpy(), dd.decdec_pack_residual_int(q_ref, rbits))


@pytest.mark.parametrize("rbits,K,N", [(8, 1, 16), (8, 127, 48), (4, 128, 1024), (4, 129, 1056), (2, 257, 6144), (8, 300, 1008), (8, 131, 6160)])
def test_residual_scale_search_at_its_edges(rbits, K, N):
    """Rows around a multiple of the 128 that are staged at a time, columns on both sides of the 1024 and 6144 where the
    column blocks widen, and columns whose quotients by a candidate scale are exact half-integers: equal to the oracle's bits."""
    g = np.random.default_rng([78, rbits, K, N])
    R32 = (g.standard_normal((K, N)) * np.exp2(g.uniform(-30, 8, N))).astype(np.float32)
    qmax = 2 ** (rbits - 1) - 1
    for n in range(0, N, 5):  # column maximum a power of two times qmax: S = that power at alpha = 1, ties at every half
        p = np.float32(2.0 ** g.integers(-18, 6))
        R32[:, n] = (g.integers(-2 * qmax, 2 * qmax + 1, K) * np.float32(0.5)) * p
        R32[0, n] = qmax * p
    R32[:, 7] = 0.0
    q_ref, S_ref = oracle.quantize_residual_sym(R32.astype(np.float64), rbits)
    codes = torch.zeros((K, N * rbits // 8), dtype=torch.uint8, pin_memory=True)
    S = torch.zeros(N, dtype=torch.float16, device="cuda")
    dd.decdec_quantize_residual(K, N, rbits, torch.from_numpy(R32).cuda(), codes, S)
    torch.cuda.synchronize()
    assert np.array_equal(S.cpu().numpy().view(np.uint16), S_ref.view(np.uint16))
    assert np.array_equal(codes.numpy(), dd.decdec_pack_residual_int(q_ref, rbits))


@pytest.mark.parametrize("rbits,K,N", [(4, 383, 64), (4, 384, 64), (4, 2049, 64), (4, 1000, 2048), (2, 3000, 2112), (8, 1500, 2112), (8, 4095, 64), (8, 4096, 64), (8, 4999, 2112), (4, 262143, 32), (4, 262144, 32)])
def test_residual_scale_search_by_bounds(rbits, K, N):
    """Each width of the column blocks, both sides of the row counts between which most candidates are ruled out beforehand, and
    columns whose values crowd a few bins of the histogram or leave many candidates equal or nearly so: the oracle's bits."""
    g = np.random.default_rng([80, rbits, K, N])
    R32 = (g.uniform(-1, 1, (K, N)) * np.exp2(g.uniform(-12, 0, N))).astype(np.float32)
    R32[:, 0::8] = g.standard_normal((K, len(range(0, N, 8)))) * 3e-3
    R32[:, 1::8] = g.laplace(size=(K, len(range(1, N, 8)))) * 1e-3
    R32[:, 2::8] = np.float32(0.75) * g.integers(-1, 2, (K, len(range(2, N, 8))))   # one magnitude: one bin
    R32[:, 3::16] = np.where(g.random((K, len(range(3, N, 16)))) < 4 / K, 1.0, 0.0)  # almost all zero
    R32[:, 4::16] = g.integers(-7, 8, (K, len(range(4, N, 16)))) * np.float32(2.0 ** -9)  # zero error at alpha = 1 with 4 bits
    R32[:, 5::16] = np.float32(3e-7) * g.standard_normal((K, len(range(5, N, 16))))  # subnormal scales, many of them the same
    R32[:, 6::16] = np.where(g.random((K, len(range(6, N, 16)))) < 0.01, g.standard_normal((K, len(range(6, N, 16)))), 1e-4)
    q_ref, S_ref = oracle.quantize_residual_sym(R32.astype(np.float64), rbits)
    codes = torch.zeros((K, N * rbits // 8), dtype=torch.uint8, pin_memory=True)
    S = torch.zeros(N, dtype=torch.float16, device="cuda")
    dd.decdec_quantize_residual(K, N, rbits, torch.from_numpy(R32).cuda(), codes, S)
    torch.cuda.synchronize()
    assert np.array_equal(S.cpu().numpy().view(np.uint16), S_ref.view(np.uint16))
    assert np.array_equal(codes.numpy(), dd.decdec_pack_residual_int(q_ref, rbits))


@pytest.mark.parametrize("rbits", [2, 4, 8])
def test_residual_columns_that_are_not_finite_get_scale_one(rbits):
    """An infinity or a NaN makes a column's error a NaN for every candidate scale; columns of large finite values, whose
    greater candidates round to an infinite scale, keep the finite ones: as in the oracle."""
    K, N = 130, 64
    R32 = np.random.default_rng([79, rbits]).standard_normal((K, N)).astype(np.float32)
    R32[:, 0] = np.inf
    R32[:, 1] = -np.inf
    R32[::2, 2] = np.inf
    R32[1::2, 2] = -np.inf
    R32[K - 1, 3] = np.inf
    R32[0, 4] = np.nan
    R32[:, 5] = np.nan
    R32[:, 6] *= 6e4 * (2 ** (rbits - 1) - 1)
    with np.errstate(invalid="ignore", over="ignore"):
        q_ref, S_ref = oracle.quantize_residual_sym(R32.astype(np.float64), rbits)
    assert np.all(S_ref[:6] == 1) and np.isfinite(S_ref[6])
    q_ref[np.isnan(R32)] = 0
    codes = torch.zeros((K, N * rbits // 8), dtype=torch.uint8, pin_memory=True)
    S = torch.zeros(N, dtype=torch.float16, device="cuda")
    dd.decdec_quantize_residual(K, N, rbits, torch.from_numpy(R32).cuda(), codes, S)
    torch.cuda.synchronize()
    assert np.array_equal(S.cpu().numpy().view(np.uint16), S_ref.view(np.uint16))
    per = 8 // rbits
    whole = ~np.isnan(R32).reshape(K, -1, per).any(axis=2)  # a NaN has no code: bytes without one
    assert np.array_equal(codes.numpy()[whole], dd.decdec_pack_residual_int(q_ref, rbits)[whole])


@pytest.mark.parametrize("rbits", [4, 2, 8])
def test_uniform_linear_with_integer_residuals_end_to_end(rbits):
    """Device-prepared layer (quantiser, fp32 residual, residual quantiser) through the hot path,
    against the oracle run on the oracle's own artefacts of the same W."""
    K, N, bits, k = 1024, 512, 3, 40
    W = workloads.weights(77, 0, 0, K, N)
    lin = UniformLinear(W, bits, rbits=rbits)
    codes, s, z = oracle.quantize_uniform(W, bits)
    W_hat = oracle.dequantize_uniform(codes, s, z)
    q_ref, S_ref = oracle.quantize_residual_sym(_residual_f32_reference(W, W_hat).astype(np.float64), rbits)
    assert np.array_equal(lin.R.numpy(), dd.decdec_pack_residual_int(q_ref, rbits))
    assert np.array_equal(lin.R_scales.cpu().numpy().view(np.uint16), S_ref.view(np.uint16))
    x = workloads.x_gauss_outliers(77, 0, 0, 0, K)
    sc = oracle.topk_abs(x, k)
    y_ref = oracle.compensated_gemv(W_hat, x, oracle.dequantize_residual_int4(q_ref, S_ref), sc)
    ws = dd.Workspace(K, N, k)
    try:
        y = torch.empty(N, dtype=torch.float16, device="cuda")
        lin.gemv(torch.from_numpy(x).cuda(), k, y, ws)
        torch.cuda.synchronize()
        assert np.array_equal(ws.read_selection(k)[0], sc)
        assert oracle.error_metric(y.cpu().numpy().astype(np.float64), y_ref) <= 2e-3
    finally:
        ws.close()
