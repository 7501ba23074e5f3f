"""Batched products against one product at a time, and 17 to 64 tokens as 16-token blocks of the streaming kernel: grids that are rounded to a multiple of eight workgroups per
block and grids that are not, one and several K ranges, n-tile counts that do not divide among the workgroups."""
import pytest

torch = pytest.importorskip("torch")

from test_gpu_mid_edges import _check  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("asym", [False, True])
@pytest.mark.parametrize("M,K,N,G", [(17, 640, 272, 128), (33, 1024, 4096, 128), (33, 1152, 4112, 0), (48, 2048, 5120, 128),
                                     (33, 11008, 1040, 0), (40, 9216, 2064, 128), (48, 1024, 16400, 0), (64, 512, 336, 0)])
def test_token_blocks(M, K, N, G, asym):
    _check(M, K, N, G, asym, ydtype="bf16" if M == 40 else "f16", hook=N < 2000)


# problems with weights of their own on grids that are not rounded: every one is the product that it is alone
@pytest.mark.parametrize("batch,M,K,N,G", [(7, 1, 1024, 1040, 0), (12, 16, 640, 272, 128), (3, 5, 1024, 4096, 256), (20, 1, 4096, 208, 0)])
def test_batched_equals_single(batch, M, K, N, G):
    import paper_2311_05161_amd as lib
    g = torch.Generator(device="cuda").manual_seed(batch + N)
    W = torch.randn((batch * N, K), generator=g, device="cuda").half()
    X = torch.randn((batch * M, K), generator=g, device="cuda").half()
    codes, step, zero = lib.quantize_weight_dint4(W, None, G)
    Xq, sx = lib.quantize_act_int8(X)
    Y = lib.w4a8_gemm_batched(Xq, sx, lib.pack_dint4(codes), step, zero, batch, M, N, K, G)
    for b in range(batch):
        r, n = slice(b * M, (b + 1) * M), slice(b * N, (b + 1) * N)
        one = lib.w4a8_gemm(Xq[r].contiguous(), sx[r].contiguous(), lib.pack_dint4(codes[n].contiguous()), step[n].contiguous(),
                            zero[n].contiguous(), N, K, G)
        assert torch.equal(Y[r], one)
