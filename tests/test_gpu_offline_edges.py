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
