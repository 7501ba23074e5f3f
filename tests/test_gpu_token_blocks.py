"""17 to 64 tokens as 16-token blocks of the streaming kernel: grids that are rounded to a multiple of eight workgroups per
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
