"""w4a8_linear on at most 16 tokens of fp16 activations and tiled weights whose K is one range of the streaming kernel: one launch
that needs no workspace and leaves one that it is given alone (several streams may have handed in the same)."""
import pytest

torch = pytest.importorskip("torch")

from test_gpu_native_calls import _layer  # noqa: E402

pytestmark = pytest.mark.gpu


# the largest K with groups and per channel, five to seven k-tiles per wave, one n-tile per workgroup and rings, up to four tokens and more
@pytest.mark.parametrize("K,N,G", [(4096, 4112, 128), (5120, 48, 128), (5120, 5136, 128), (5120, 272, 256), (5248, 80, 0),
                                   (6144, 4112, 0), (7168, 4112, 0)])
@pytest.mark.parametrize("M", [4, 5, 16])
def test_one_launch_leaves_the_workspace_alone(M, K, N, G):
    import paper_2311_05161_amd as w
    X, s, Wp, step, zero, _ = _layer(M, K, N, G)
    need = int(w.load_library().w4a8_linear_workspace_bytes(M, N, K, G, w.LAYOUT_TILED))
    ws = torch.full((need + 4096,), 0xa5, dtype=torch.uint8, device="cuda")
    Y = w.w4a8_linear(X, s, Wp, step, zero, N, G, workspace=ws)
    assert bool((ws == 0xa5).all())
    for got in (w.w4a8_linear(X, s, Wp, step, zero, N, G),                                             # fresh outputs only
                w.w4a8_gemm(*w.quantize_act_int8(X, s), Wp, step, zero, N, K, G)):
        assert torch.equal(got, Y)
    c = w.load_library()
    Y2 = torch.empty_like(Y)
    st = torch.cuda.current_stream().cuda_stream
    assert c.w4a8_linear(X.data_ptr(), 1, M, K, K, s.data_ptr(), Wp.data_ptr(), 1, step.data_ptr(), zero.data_ptr(), N, G,
                         Y2.data_ptr(), 1, N, None, None, None, None, 0, st) == 0                      # no workspace at all
    assert torch.equal(Y2, Y)
