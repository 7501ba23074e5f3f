"""Everywhere but on the streaming kernel, whose waves share the k-tiles of a group, the integer sum of a whole group is rounded once:
activations whose k-tiles cancel inside every group (against weights that repeat from k-tile to k-tile) give exact zeros, where sums
rounded k-tile by k-tile leave rests."""
import pytest

torch = pytest.importorskip("torch")

from test_launch_plans import route  # noqa: E402

pytestmark = pytest.mark.gpu


# K in phases inside the workgroup (tiles of two to four token blocks, four phases and two, phases without a group in the last
# round, few groups, and groups that are halves of K), K in ranges over workgroups, decoded weights
@pytest.mark.parametrize("M,K,N,G,form", [
    (129, 3072, 1040, 256, (4, 2)), (209, 4352, 2048, 256, (4, 2)), (300, 1536, 6160, 384, (2, 2)), (50, 3840, 21520, 640, (2, 2)),
    (300, 1152, 6160, 384, (2, 2)), (233, 4096, 1632, 1024, (4, 2)), (300, 8192, 1040, 4096, (2, 2)), (143, 6144, 2112, 2048, None), (513, 3072, 4112, 512, (2, 3)), (502, 12288, 3120, 1024, (4, 4)), (200, 5120, 13824, 256, (2, 4)),
    (150, 8192, 2064, 1024, None), (2048, 3072, 4096, 512, None), (2048, 5120, 13824, 256, None)])
@pytest.mark.parametrize("asym", [False, True])
def test_whole_groups_are_rounded_once(M, K, N, G, form, asym):
    import paper_2311_05161_amd as w
    if not asym:
        r = route(M, K, N, G)
        assert r[1:] == form if form else r[0] == "tile"
    g = torch.Generator(device="cuda").manual_seed(K + N)
    T = G // 128
    a, b = (torch.randint(-60, 61, (M, K // G, 128), generator=g, device="cuda") for _ in "ab")
    X = torch.zeros((M, K // G, T, 128), dtype=torch.int64, device="cuda")
    X[:, :, 0], X[:, :, T - 1] = a, -a      # two k-tiles that cancel, or (what shows the rounding of single ones best) three
    if T > 2:
        X[:, :, 1], X[:, :, T - 1] = b, -(a + b)
    Xq = X.reshape(M, K).to(torch.int8).contiguous()
    codes = torch.randint(0, 16, (N, K // G, 1, 128), generator=g, device="cuda").expand(N, K // G, T, 128)
    codes = codes.reshape(N, K).to(torch.uint8).contiguous()
    zero = torch.randint(0, 14, (N, K // G), generator=g, device="cuda", dtype=torch.uint8)
    step = torch.rand((N, K // G), generator=g, device="cuda") * 0.9 + 0.1
    sx = torch.full((M,), 1e3, device="cuda")   # (a rest of one rounding is far above the smallest fp16 number)
    Wp = w.pack_dint4(codes)
    if asym:   # zero-points of zero: the same sums through the other instances
        wsum, tsum = w.dint4_weight_sums(codes, zero, G)
        zx = torch.zeros((M,), dtype=torch.int32, device="cuda")
        Y = w.w4a8_gemm_asym(Xq, sx, zx, Wp, step, zero, wsum, tsum, N, K, G)
    else:
        Y = w.w4a8_gemm(Xq, sx, Wp, step, zero, N, K, G)
    assert int((Y != 0).sum()) == 0
