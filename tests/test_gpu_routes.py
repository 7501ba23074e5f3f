"""Every form of the group-wise kernels at shapes that leave rests everywhere (a last token tile that is not full, channels that end
inside a workgroup, phases without a group in the last round), with and without the accumulator hook, on the kernel that is meant."""
import pytest

pytest.importorskip("torch")

from test_gpu_mid_edges import _check  # noqa: E402
from test_launch_plans import route  # noqa: E402

# M, K, N, G, token zero-points, (phases, token blocks)
FORMS = [
    (109, 1152, 9296, 128, False, (2, 2)), (136, 1152, 11488, 128, False, (2, 3)), (195, 1664, 11200, 128, False, (2, 4)),
    (182, 1152, 336, 128, False, (4, 2)), (73, 1152, 8912, 128, False, (4, 3)), (102, 2176, 8464, 128, False, (4, 4)),
    (109, 1152, 9296, 128, True, (2, 2)), (136, 1152, 11488, 128, True, (2, 3)), (195, 1664, 11200, 128, True, (2, 4)),
    (182, 1152, 336, 128, True, (4, 2)), (69, 1152, 9584, 128, True, (4, 3)), (367, 1152, 5392, 128, True, (4, 4)),
    # groups of several k-tiles
    (133, 1152, 352, 384, False, (2, 2)), (137, 1152, 11376, 384, False, (2, 3)), (196, 1152, 11936, 384, False, (2, 4)),
    (154, 1280, 368, 256, False, (4, 2)), (69, 1152, 9232, 384, False, (4, 3)), (106, 1920, 8752, 640, False, (4, 4)),
    (133, 1152, 352, 384, True, (2, 2)), (137, 1152, 11376, 384, True, (2, 3)), (154, 1280, 368, 256, True, (4, 2)),
    (69, 1152, 11936, 384, True, (4, 3)), (513, 3072, 4112, 512, True, (2, 3)), (645, 4608, 2016, 512, False, (4, 3))]
# the tile kernel: 64 rows, K in ranges in groups of one, three and four k-tiles
TILES = [(63, 3328, 36944, 128, 64, 1), (149, 8448, 1072, 384, 128, 11), (1021, 6656, 80, 128, 128, 13), (361, 4608, 912, 512, 128, 9)]


@pytest.mark.parametrize("M,K,N,G,asym,form", FORMS)
def test_forms(M, K, N, G, asym, form):
    assert route(M, K, N, G, asym) == ("phases", *form)


@pytest.mark.parametrize("asym", [False, True])
@pytest.mark.parametrize("M,K,N,G,rows,ranges", TILES)
def test_tiles(M, K, N, G, rows, ranges, asym):
    assert route(M, K, N, G, asym) == ("tile", rows, ranges, 0)


@pytest.mark.gpu
@pytest.mark.parametrize("M,K,N,G,asym,form", FORMS)
def test_products_of_forms(M, K, N, G, asym, form):
    _check(M, K, N, G, asym, ydtype="bf16" if M % 2 else "f16", ypad=1)
    _check(M, K, N, G, asym, hook=True)


@pytest.mark.gpu
@pytest.mark.parametrize("asym", [False, True])
@pytest.mark.parametrize("M,K,N,G,rows,ranges", TILES)
def test_products_of_tiles(M, K, N, G, rows, ranges, asym):
    _check(M, K, N, G, asym, hook=ranges > 1)
    if ranges > 1:
        _check(M, K, N, G, asym)
