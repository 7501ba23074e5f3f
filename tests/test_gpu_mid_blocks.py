"""The K-phase kernel on tiles of two, three and four token blocks, four phases and two: ragged token tiles (a row beyond whole
ones, one short of them), channels that end inside a workgroup, k-tile counts that leave phases idle, with and without token
zero-points."""
import ctypes

import pytest

pytest.importorskip("torch")

from test_gpu_mid_edges import _check  # noqa: E402
from test_launch_plans import I64, MidForm, _rule  # noqa: E402


def form(M, K, N, asym=False):
    r = _rule("13gemm_mid_formEllllb", MidForm, I64, I64, I64, I64, ctypes.c_bool)(M, N, K, 128, asym)
    return (r.phases, r.blocks) if r.phases else None


SHAPES = [(64, 1152, 16336, (4, 2)), (129, 1408, 1040, (4, 2)), (191, 1280, 2064, (4, 2)), (257, 1152, 1360, (4, 2)),
          (50, 1024, 21520, (2, 2)), (385, 1024, 4112, (2, 2)), (300, 1152, 6160, (2, 2)),
          (190, 4096, 8176, (4, 3)), (289, 4992, 3600, (4, 3)),
          (129, 1536, 13824, (2, 3)), (513, 1664, 4112, (2, 3)), (671, 1408, 4080, (2, 3)),
          (500, 3968, 4096, (4, 4)), (1024, 1792, 4096, (2, 4)), (200, 1664, 13776, (2, 4))]


@pytest.mark.parametrize("M,K,N,want", SHAPES)
def test_forms(M, K, N, want):
    assert form(M, K, N) == want


# one shape on either side of each line between the kernels (the times stand beside the rule)
@pytest.mark.parametrize("M,K,N,want", [
    (607, 4096, 4096, (2, 3)), (524, 7936, 1024, (4, 2)), (59, 9856, 15712, (4, 2)), (113, 4224, 6496, (4, 2)),
    (62, 7296, 2960, None), (32, 2048, 5344, None), (316, 9728, 16384, None), (1200, 4096, 8192, None), (607, 640, 4096, None)])
def test_lines(M, K, N, want):
    assert form(M, K, N) == want


@pytest.mark.gpu
@pytest.mark.parametrize("asym", [False, True])
@pytest.mark.parametrize("M,K,N,want", SHAPES)
def test_products(M, K, N, want, asym):
    _check(M, K, N, 128, asym, ydtype="bf16" if M % 2 else "f16", ypad=M % 3)


# groups of several k-tiles: a phase has whole ones (the last shape would otherwise be token blocks, whose
# workspace holds no partial sums)
@pytest.mark.gpu
@pytest.mark.parametrize("asym", [False, True])
@pytest.mark.parametrize("M,K,N,G", [(129, 1536, 1040, 256), (300, 1152, 6160, 384), (513, 2560, 4112, 512), (50, 1280, 21520, 640)])
def test_larger_groups(M, K, N, G, asym):
    r = _rule("13gemm_mid_formEllllb", MidForm, I64, I64, I64, I64, ctypes.c_bool)(M, N, K, G, asym)
    assert r.phases > 0
    _check(M, K, N, G, asym)
    if M < 200:
        _check(M, K, N, G, asym, hook=True)


@pytest.mark.gpu
@pytest.mark.parametrize("M,K,N", [(129, 1408, 1040), (300, 1152, 1360), (385, 1024, 1552)])
def test_accumulators(M, K, N):
    for asym in (False, True):
        assert form(M, K, N, asym) is not None
        _check(M, K, N, 128, asym, hook=True)
