"""Edges of the activation quantizers: row counts and lengths at which another kernel or instance is taken, and the row-sums
that the one-call layer takes from the quantizer."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import synthetic_inputs as syn  # noqa: E402
from gpu_util import acc_by_float64_matmul, assert_y_close, decode_table_np, dev, host  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lib():
    import paper_2311_05161_amd as w
    w.load_library()
    return w


# 256 / 257 rows and 2040 / 2048 columns (with 128 / 129 rows) are the edges of the workgroup-per-row form, 8192 / 8200 those of
# its two instances, 16384 the longest row of the vector kernels
@pytest.mark.parametrize("M,K", [(1, 2040), (1, 2048), (128, 2048), (129, 2048), (256, 2056), (257, 2056), (7, 8192), (7, 8200), (3, 16384), (2, 16392)])
@pytest.mark.parametrize("dtype", ["f16", "bf16", "f32"])
def test_act_quant_row_edges(lib, oracle, M, K, dtype):
    X, _, s = syn.random_layer(M + K, M, K, 16, x_dtype="f32")
    Xd = dev(X).to({"f16": torch.float16, "bf16": torch.bfloat16, "f32": torch.float32}[dtype])
    Xd[-1] = 0.0 if M > 1 else Xd[-1]
    for scale in (s, None):
        Xq, sx = lib.quantize_act_int8(Xd, None if scale is None else dev(scale))
        q, r = oracle.quantize_act_int8(Xd.float().cpu().numpy(), scale)
        assert np.array_equal(host(Xq), q) and np.array_equal(host(sx).view(np.uint32), r.view(np.uint32))
        Aq, ax, az = lib.quantize_act_int8_asym(Xd, None if scale is None else dev(scale))
        q, r, z = oracle.quantize_act_uint8_asym(Xd.float().cpu().numpy(), scale)
        assert np.array_equal(host(Aq).astype(np.int32) + 128, q.astype(np.int32))
        assert np.array_equal(host(ax).view(np.uint32), r.view(np.uint32)) and np.array_equal(host(az) + 128, z)


# per-channel layers that read row-sums: the K-phase kernel, both tile kernels, a tile kernel with its last channels on the
# K-phase kernel (both read the same sums), K in ranges (which makes its own) and rows that the vector quantizer does not take
# (pre-pass)
@pytest.mark.parametrize("M,K,N,pad", [(130, 2048, 272, 0), (300, 2560, 528, 0), (700, 1024, 4112, 8), (270, 5248, 16, 0),
                                       (2100, 256, 8208, 0), (140, 2048, 256, 3), (1100, 3072, 14480, 0),
                                       (3495, 3072, 4656, 8)])
def test_row_sums_from_the_quantizer(lib, oracle, M, K, N, pad):
    X, W, s = syn.random_layer(M + N, M, K, N)
    buf = torch.zeros((M, K + pad), dtype=torch.float16, device="cuda")
    buf[:, :K] = dev(X)
    codes, step, zero = lib.quantize_weight_dint4(dev(W), dev(s), 0)
    Wp = lib.pack_dint4(codes)
    Y, Xq, sx = lib.w4a8_linear(buf[:, :K], dev(s), Wp, step, zero, N, want_quantized=True)
    Xq2, sx2 = lib.quantize_act_int8(buf[:, :K], dev(s))
    assert torch.equal(Xq, Xq2) and torch.equal(sx, sx2)
    assert torch.equal(Y, lib.w4a8_gemm(Xq2, sx2, Wp, step, zero, N, K))   # which sums the rows itself
    rows = np.unique(np.linspace(0, M - 1, 40).astype(int))
    acc = acc_by_float64_matmul(host(Xq)[rows], decode_table_np(host(codes), host(zero), 0), 0)[..., 0]
    assert_y_close(host(Y)[rows], host(sx)[rows].astype(np.float64)[:, None] * acc * (host(step).astype(np.float64)[:, 0] / 2))
