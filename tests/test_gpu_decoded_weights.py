"""Group-wise products on weights decoded to int8 beforehand: the same bits as on the packed weights, which a workspace
without room for the decoded ones still gets."""
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


# ragged last tiles of tokens and channels (N % 32 = 16), groups of several k-tiles, an odd number of k-tiles, the last round of tiles
# with K in ranges, outputs that allow 16-byte, 8-byte and 2-byte stores, all levels of plain INT4
@pytest.mark.parametrize("M,K,N,G,fmt,y,pad", [
    (4200, 3072, 1008, 128, 0, "f16", 0), (4224, 3200, 1024, 128, 0, "bf16", 4), (4200, 6144, 1008, 384, 0, "f16", 1),
    (4104, 5120, 2032, 128, 0, "f16", 0), (4104, 5120, 2032, 256, 1, "bf16", 2), (8200, 2816, 528, 128, 1, "f16", 8)])
def test_same_bits_as_packed(M, K, N, G, fmt, y, pad):
    import paper_2311_05161_amd as w
    lib = w.load_library()
    g = torch.Generator(device="cuda").manual_seed(M + N)
    Xq = torch.randint(-127, 128, (M, K), generator=g, device="cuda", dtype=torch.int8)
    sx = torch.rand((M,), generator=g, device="cuda") + 0.01
    step = torch.rand((N, K // G), generator=g, device="cuda") + 0.01
    zero = torch.randint(0, 16 if fmt else 14, (N, K // G), generator=g, device="cuda", dtype=torch.uint8)
    Wp = torch.randint(0, 256, (N * K // 2,), generator=g, device="cuda", dtype=torch.uint8)   # every nibble is a code
    full = int(lib.w4a8_gemm_workspace_preferred_bytes(M, N, K, G, 1))
    decoded = (N + 31) // 32 * 32 * K + K // 128 * ((N + 255) // 256 * 256) * 4
    assert full - decoded == int(lib.w4a8_gemm_workspace_bytes(M, N, K, G, 1))   # the shape takes the route
    out = []
    for need in (full, full - decoded):
        ws = torch.full((max(need, 1),), 255, dtype=torch.uint8, device="cuda")
        Y = torch.full((M, N + pad), 7.0, dtype=torch.float16 if y == "f16" else torch.bfloat16, device="cuda")
        assert lib.w4a8_gemm_format(Xq.data_ptr(), sx.data_ptr(), M, Wp.data_ptr(), 1, step.data_ptr(), zero.data_ptr(), N, K, G,
                                    fmt, Y.data_ptr(), 1 if y == "f16" else 2, N + pad, None, ws.data_ptr(), need,
                                    torch.cuda.current_stream().cuda_stream) == 0
        out.append(Y.view(torch.int16))
    assert torch.equal(out[0], out[1])
    if pad:
        assert (out[0][:, N:] == torch.full((), 7.0, dtype=Y.dtype).view(torch.int16).item()).all()


# a product that needs no workspace takes one that lies anywhere, also where it would decode the weights into an aligned one
@pytest.mark.parametrize("offset", [0, 8, 64])
def test_workspace_off_the_alignment(offset):
    import paper_2311_05161_amd as w
    lib = w.load_library()
    M, K, N, G = 4096, 3072, 2048, 128
    g = torch.Generator(device="cuda").manual_seed(3)
    Xq = torch.randint(-127, 128, (M, K), generator=g, device="cuda", dtype=torch.int8)
    sx, step = torch.rand((M,), generator=g, device="cuda"), torch.rand((N, K // G), generator=g, device="cuda")
    zero = torch.randint(0, 14, (N, K // G), generator=g, device="cuda", dtype=torch.uint8)
    Wp = torch.randint(0, 256, (N * K // 2,), generator=g, device="cuda", dtype=torch.uint8)
    need = int(lib.w4a8_gemm_workspace_preferred_bytes(M, N, K, G, 1))
    assert need > 0 and int(lib.w4a8_gemm_workspace_bytes(M, N, K, G, 1)) == 0
    ws = torch.empty((need + 256,), dtype=torch.uint8, device="cuda")
    out = []
    for p, size in ((ws.data_ptr() + offset, need), (None, 0)):
        Y = torch.empty((M, N), dtype=torch.float16, device="cuda")
        assert lib.w4a8_gemm(Xq.data_ptr(), sx.data_ptr(), M, Wp.data_ptr(), 1, step.data_ptr(), zero.data_ptr(), N, K, G,
                             Y.data_ptr(), 1, N, None, p, size, torch.cuda.current_stream().cuda_stream) == 0
        out.append(Y)
    assert torch.equal(out[0], out[1])
