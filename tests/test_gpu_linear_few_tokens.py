"""The one-launch decode step at one to five tokens: up to four, the in-launch quantizer spreads its lanes over four rows."""
import pytest

torch = pytest.importorskip("torch")

from test_gpu_parity_linear import _case, lib  # noqa: E402,F401

pytestmark = pytest.mark.gpu

# k-tiles per wave 1, 2, 3, 4, 5 (groups) and 6, 7 (per channel), a single n-tile per workgroup and rings, ragged k-tiles
SHAPES = [(128, 16, 128), (1024, 8208, 128), (2048, 48, 256), (2944, 4112, 128), (4096, 4096, 128), (5120, 4624, 0),
          (5248, 80, 0), (6144, 4112, 0), (7168, 4112, 0)]


@pytest.mark.parametrize("K,N,G", SHAPES)
@pytest.mark.parametrize("M", [1, 2, 3, 4, 5])
def test_few_tokens(lib, oracle, M, K, N, G):  # noqa: F811
    _case(lib, oracle, 900 + M + K, M, K, N, G, pad=8 * (M % 2), use_s=M != 3)
