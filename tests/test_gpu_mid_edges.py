"""The kernels that cut K into phases inside the workgroup, at the edges of their tiles, phase counts and dispatch rule:
token counts around 128-row tiles, channels that end inside a workgroup, k-tile counts that leave phases idle, both phase
counts, with and without token zero-points, and the neighbouring shapes that the tile kernel takes."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from gpu_util import acc_by_float64_matmul, assert_y_close, decode_table_np, dev, host  # noqa: E402

pytestmark = pytest.mark.gpu


def _check(M, K, N, G, asym, ydtype="f16", ypad=0, fmt=0, hook=False):
    import paper_2311_05161_amd as lib
    rng = np.random.default_rng(M * 7 + K + N)
    ng = K // (G or K)
    Xq = rng.integers(-128 if asym else -127, 128, (M, K), dtype=np.int8)
    sx = rng.uniform(0.01, 0.02, M).astype(np.float32)
    zx = rng.integers(-128, 128, M, dtype=np.int32)
    codes = rng.integers(0, 16, (N, K), dtype=np.uint8)
    step = rng.uniform(0.001, 0.002, (N, ng)).astype(np.float32)
    zero = rng.integers(0, 14, (N, ng), dtype=np.uint8)
    yt = torch.float16 if ydtype == "f16" else torch.bfloat16
    Y = torch.full((M, N + ypad), -1.0, dtype=yt, device="cuda")
    cd, zd = dev(codes), dev(zero)
    args = (lib.pack_dint4(cd), dev(step), zd)
    acc_gpu = torch.empty((M, N, ng), dtype=torch.int32, device="cuda") if hook else None
    if asym:
        ws, ts = lib.dint4_weight_sums(cd, zd, G)
        lib.w4a8_gemm_asym(dev(Xq), dev(sx), dev(zx), *args, ws, ts, N, K, G, Y=Y[:, :N], acc_out=acc_gpu)
    else:
        lib.w4a8_gemm(dev(Xq), dev(sx), *args, N, K, G, Y=Y[:, :N], acc_out=acc_gpu)
    X = Xq.astype(np.int32) - (zx[:, None] if asym else 0)
    acc = acc_by_float64_matmul(X, decode_table_np(codes, zero, G), G)
    y64 = sx.astype(np.float64)[:, None] * (acc * (step.astype(np.float64) / 2)).sum(2)
    assert_y_close(host(Y[:, :N].contiguous()), y64, ydtype)
    if ypad:
        assert (host(Y[:, N:].contiguous()) == -1.0).all()
    if hook:
        assert np.array_equal(host(acc_gpu), acc.astype(np.int64))


# Where the four-block form has four phases: 64 .. 256 workgroups of 64 channels; 9, 10, 11, 13 k-tiles leave phases without one in the
# last step (which form each shape gets: test_launch_plans.py; every form at its ragged edges: test_gpu_routes.py)
FOUR = [(65, 1024, 4096), (257, 1152, 1360), (300, 1280, 1360), (385, 1408, 1040), (512, 1664, 4096), (1000, 1024, 1040)]
# where it has two: more than 256 of those, up to 256 of 128 channels; odd and even counts of k-tiles
TWO = [(129, 1536, 13824), (513, 1664, 4112), (640, 2048, 4096), (1024, 1792, 4096), (2048, 1536, 2032)]
# few workgroups and long K (two or three token blocks by now), four phases over 128 k-tiles, and what stays on the tile kernel: few
# k-tiles, too many workgroups
TILE = [(300, 2048, 512), (600, 16384, 1040), (600, 16384, 2560), (1024, 1024, 4096), (1100, 1536, 4096), (2048, 1536, 2064)]


@pytest.mark.parametrize("asym", [False, True])
@pytest.mark.parametrize("M,K,N", FOUR + TWO + TILE)
def test_group_128(M, K, N, asym):
    _check(M, K, N, 128, asym)


@pytest.mark.parametrize("M,K,N", [FOUR[1], TWO[1]])
def test_group_128_hook_and_rows_off_alignment(M, K, N):
    for asym in (False, True):
        _check(M, K, N, 128, asym, hook=True)
    _check(M, K, N, 128, True, ydtype="bf16", ypad=1)


# per channel: beyond 256 tokens, the last K that it takes there and the first that it leaves
@pytest.mark.parametrize("M,K,N", [(257, 1024, 272), (1000, 1152, 1024), (4096, 1024, 256), (300, 9216, 528), (300, 9344, 528)])
def test_per_channel(M, K, N):
    _check(M, K, N, 0, False)
    if M < 400:
        _check(M, K, N, 0, False, hook=True)


# per channel, a few tiles beyond a whole round of 512: from K = 3072 the last channels (one ragged 64-channel part and more,
# few and many token tiles) go to the K-phase kernel; with zero-points or the accumulator hook the whole layer stays on the tile
# kernel and gives the same outputs.  (4140, 3072, 4112) has too many such channels, the short K stay whole.
@pytest.mark.parametrize("M,K,N", [(1100, 3072, 14480), (1100, 3200, 14592), (3495, 3072, 4656), (4140, 3072, 4112),
                                   (1100, 1024, 14480), (1100, 1152, 14592), (4140, 1024, 4112)])
def test_per_channel_remainder(M, K, N):
    import paper_2311_05161_amd as lib
    _check(M, K, N, 0, False, ypad=3)
    if K in (1024, 3072) and N > 10000:
        _check(M, K, N, 0, True)
    rng = np.random.default_rng(5)
    Xq = dev(rng.integers(-127, 128, (M, K), dtype=np.int8))
    sx = dev(rng.uniform(0.01, 0.02, M).astype(np.float32))
    codes = dev(rng.integers(0, 16, (N, K), dtype=np.uint8))
    step, zero = torch.rand((N, 1), device="cuda") * 0.01, torch.full((N, 1), 5, dtype=torch.uint8, device="cuda")
    Wp = lib.pack_dint4(codes)
    Y, _ = lib.w4a8_gemm(Xq, sx, Wp, step, zero, N, K, 0, want_acc=True)
    assert torch.equal(Y, lib.w4a8_gemm(Xq, sx, Wp, step, zero, N, K, 0))


# token zero-points at the ends of their range against the largest weight sums of a group, where what leaves the accumulators in
# binary32 is largest: products up to 128 * 104 * 128 (below 2^21), sums with them up to 255 * 104 * 128 (below 2^22), both exact
@pytest.mark.parametrize("M,K,N", [FOUR[0], TWO[0], (607, 1024, 4096), (97, 2048, 4112)])
@pytest.mark.parametrize("code,z", [(13, 0), (0, 13), (12, 0)])
def test_zero_points_at_the_ends(M, K, N, code, z):
    import paper_2311_05161_amd as lib
    Xq = np.full((M, K), 127, np.int8)
    Xq[::2] = -128
    Xq[::3, ::7] = -127
    zx = np.where(np.arange(M) % 4 < 2, -128, 127).astype(np.int32)
    sx = np.full(M, 0.01, np.float32)
    codes = np.full((N, K), code, np.uint8)
    codes[::5, ::9] = 14
    zero = np.full((N, K // 128), z, np.uint8)
    step = np.full((N, K // 128), 1e-5, np.float32)
    cd, zd = dev(codes), dev(zero)
    ws, ts = lib.dint4_weight_sums(cd, zd, 128)
    Y = torch.empty((M, N), dtype=torch.float16, device="cuda")
    lib.w4a8_gemm_asym(dev(Xq), dev(sx), dev(zx), lib.pack_dint4(cd), dev(step), zd, ws, ts, N, K, 128, Y=Y)
    acc = acc_by_float64_matmul(Xq.astype(np.int32) - zx[:, None], decode_table_np(codes, zero, 128), 128)
    assert_y_close(host(Y), sx.astype(np.float64)[:, None] * (acc * (step.astype(np.float64) / 2)).sum(2), "f16")
