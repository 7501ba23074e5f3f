"""Edges of the offline kernels: sizes, group lengths and alignments at which another branch or instance is taken."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import synthetic_inputs as syn  # noqa: E402
from gpu_util import decode_table_np, dev, host, tiled_layout_np  # noqa: E402,F401

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lib():
    import paper_2311_05161_amd as w
    w.load_library()
    return w


# one group per row of every lane count (8, 16, 32, a whole wave with a ragged last round), a last wave that is
# partly empty, and codes that are not 16-byte aligned (the general kernel)
@pytest.mark.parametrize("N,K,G,shift", [
    (16, 128, 128, 0), (48, 1152, 128, 0), (33, 768, 256, 0), (5, 2560, 512, 0), (7, 384, 384, 0),
    (16, 1024, 0, 0), (3, 9216, 0, 0), (2, 4224, 0, 0), (16, 384, 128, 4), (5, 96, 48, 0)])
def test_weight_sums_edges(lib, N, K, G, shift):
    rng = np.random.default_rng(N * 7919 + K)
    codes = rng.integers(0, 16, (N, K), dtype=np.uint8)
    codes[0] = 14
    codes[-1, ::2] = 15
    ng = K // (G or K)
    zero = rng.integers(0, 14, (N, ng), dtype=np.uint8)
    want = decode_table_np(codes, zero, G).astype(np.int64)
    buf = torch.zeros(N * K + shift, dtype=torch.uint8, device="cuda")
    buf[shift:] = dev(codes).view(-1)
    if K % 128 == 0 and (G or K) % 128 == 0:
        wsum, tsum = lib.dint4_weight_sums(buf[shift:].view(N, K), dev(zero), G)
        assert np.array_equal(host(tsum), want.reshape(N, K // 128, 128).sum(2))
    else:
        wsum = torch.full((N, ng), -1, dtype=torch.int32, device="cuda")
        assert lib.load_library().dint4_weight_sums(buf[shift:].data_ptr(), dev(zero).data_ptr(), N, K, G,
                                                    wsum.data_ptr(), None, None) == 0
    assert np.array_equal(host(wsum), want.reshape(N, ng, -1).sum(2))


# a last block with one tile, odd tile counts, both sources and both code spaces, and buffers off the 16-byte
# alignment (the general kernel); upper bits of the code bytes are ignored
@pytest.mark.parametrize("N,K", [(16, 128), (48, 384), (80, 1152)])
@pytest.mark.parametrize("plain", [False, True])
@pytest.mark.parametrize("shift", [0, 4])
def test_pack_tiles_edges(lib, N, K, plain, shift):
    rng = np.random.default_rng(N + K)
    codes = rng.integers(0, 256, (N, K), dtype=np.uint8)
    c = codes & 15
    # ordinary INT4: codes 14 and 15 are the lower and upper member of the last pair, as dINT4's 15 and 14 are
    want = tiled_layout_np(np.where(c >= 14, c ^ 1, c) if plain else c)
    fmt = lib.FMT_INT4 if plain else lib.FMT_DINT4
    src = torch.zeros(N * K + shift, dtype=torch.uint8, device="cuda")
    src[shift:] = dev(codes).view(-1)
    dst = torch.zeros(N * K // 2 + shift, dtype=torch.uint8, device="cuda")
    c_lib = lib.load_library()
    assert c_lib.pack_format(src[shift:].data_ptr(), N, K, dst[shift:].data_ptr(), lib.LAYOUT_TILED, fmt, None) == 0
    assert np.array_equal(host(dst)[shift:], want)
    # canonical bytes re-tiled on the way into a product give what the tiled form gives
    X = dev(rng.integers(-127, 128, (3, K), dtype=np.int8))
    sx = torch.ones(3, device="cuda")
    step, zero = torch.ones((N, 1), device="cuda"), torch.full((N, 1), 5, dtype=torch.uint8, device="cuda")
    canon = torch.zeros(N * K // 2 + shift, dtype=torch.uint8, device="cuda")
    canon[:N * K // 2] = lib.pack_format(dev(c), lib.LAYOUT_CANONICAL, fmt).view(-1)
    Y = [torch.empty((3, N), dtype=torch.float16, device="cuda") for _ in range(2)]
    need = lib.gemm_workspace_bytes(3, N, K, 0, lib.LAYOUT_CANONICAL)
    ws = torch.empty(max(need, 256), dtype=torch.uint8, device="cuda")
    for layout, w, y in ((lib.LAYOUT_CANONICAL, canon, Y[0]), (lib.LAYOUT_TILED, dev(want), Y[1])):
        assert c_lib.w4a8_gemm_format(X.data_ptr(), sx.data_ptr(), 3, w.data_ptr(), layout, step.data_ptr(),
                                      zero.data_ptr(), N, K, 0, fmt, y.data_ptr(), 1, N, None, ws.data_ptr(),
                                      ws.numel(), None) == 0
    assert torch.equal(Y[0], Y[1])
