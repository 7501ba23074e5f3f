"""Products whose K is cut into ranges: the kernel that adds the ranges' partial sums, at its edges (more than four
ranges, channels that do not fill a block, rows of Y off the vector alignment, both output types, both forms, and both
sides of the 1024 blocks, 2048 with more than four ranges, up to which a thread makes one, channels in eighths for the XCDs (whole and ragged) and in row-major order)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from gpu_util import acc_by_float64_matmul, assert_y_close, decode_table_np, dev, host  # noqa: E402
from test_launch_plans import route  # noqa: E402

pytestmark = pytest.mark.gpu


# tile kernel with K in ranges: one output per thread beyond 1024 blocks, the XCDs' eighths whole and ragged, row-major order whole
# and ragged, each up to four ranges and beyond
RANGES = [(1033, 5376, 48, 128), (385, 1024, 6944, 128), (361, 4608, 912, 512), (1298, 4608, 256, 512), (153, 1280, 5888, 0),
          (149, 2304, 5760, 0), (779, 1024, 1280, 0), (586, 1024, 4752, 128), (1208, 4608, 272, 512), (1109, 1536, 48, 512)]


@pytest.mark.parametrize("M,K,N,G", RANGES)
def test_ranges_are_on_the_tile_kernel(M, K, N, G):
    r = route(M, K, N, G)
    assert r[0] == "tile" and r[2] >= 2


@pytest.mark.parametrize("M,K,N,G", [(16, 13824, 1040, 128), (3, 11008, 48, 0), (130, 16384, 48, 128),
                                     (130, 16384, 48, 0), (260, 8192, 272, 512), (1, 27648, 16, 0),
                                     (64, 11008, 4096, 0), (70, 13824, 4112, 512),
                                     (1290, 5120, 48, 128), (1030, 16384, 304, 128),
                                     (390, 5120, 1024, 256), (173, 1280, 8128, 256), (150, 2048, 2064, 512),
                                     (130, 5120, 4112, 0)] + RANGES)
@pytest.mark.parametrize("ypad,ydtype", [(0, "f16"), (1, "bf16"), (6, "f16")])
def test_combine_edges(M, K, N, G, ypad, ydtype):
    import paper_2311_05161_amd as lib
    rng = np.random.default_rng(M * 31 + K + N)
    ng = K // (G or K)
    Xq = rng.integers(-127, 128, (M, K), dtype=np.int8)
    sx = rng.uniform(0.01, 0.02, M).astype(np.float32)
    codes = rng.integers(0, 16, (N, K), dtype=np.uint8)
    step = rng.uniform(0.001, 0.002, (N, ng)).astype(np.float32)
    zero = rng.integers(0, 14, (N, ng), dtype=np.uint8)
    Y = torch.full((M, N + ypad), -1.0, dtype=torch.float16 if ydtype == "f16" else torch.bfloat16, device="cuda")
    assert lib.gemm_workspace_bytes(M, N, K, G) >= 2 * 4 * M * N      # partial sums of two ranges at least
    lib.w4a8_gemm(dev(Xq), dev(sx), lib.pack_dint4(dev(codes)), dev(step), dev(zero), N, K, G, Y=Y[:, :N])
    acc = acc_by_float64_matmul(Xq, decode_table_np(codes, zero, G), G)
    y64 = sx.astype(np.float64)[:, None] * (acc * (step.astype(np.float64) / 2)).sum(2)
    assert_y_close(host(Y[:, :N].contiguous()), y64, ydtype)
    assert (host(Y[:, N:].contiguous()) == -1.0).all()
