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


# a last block with one tile, odd tile counts, both sources and both code spaces, and buffers off the 16-byte
# alignment (the general kernel); upper bits of the code bytes are ignored
@pytest.mark.parametrize("N,K", [(16, 128), (48, 384), (80, 1152)])
@pytest.mark.parametrize("plain", [False, True])
@pytest.mark.parametrize("shift", [0, 4])
def test_pack_tiles_edges(lib, N, K, plain, shift):
    rng = np.random.default_rng(N + K)
    codes = rng.integers(0, 256, (N, K), dtype=np.uint8)
    c = codes & 15
    # ordinary INT4: codes 14 and 15 are the lower and upper member of the last pair, as dINT4's 15 and 14 are
    want = tiled_layout_np(np.where(c >= 14, c ^ 1, c) if plain else c)
    fmt = lib.FMT_INT4 if plain else lib.FMT_DINT4
    src = torch.zeros(N * K + shift, dtype=torch.uint8, device="cuda")
    src[shift:] = dev(codes).view(-1)
    dst = torch.zeros(N * K // 2 + shift, dtype=torch.uint8, device="cuda")
    c_lib = lib.load_library()
    assert c_lib.pack_format(src[shift:].data_ptr(), N, K, dst[shift:].data_ptr(), lib.LAYOUT_TILED, fmt, None) == 0
    assert np.array_equal(host(dst)[shift:], want)
    # canonical bytes re-tiled on the way into a product give what the tiled form gives
    X = dev(rng.integers(-127, 128, (3, K), dtype=np.int8))
    sx = torch.ones(3, device="cuda")
    step, zero = torch.ones((N, 1), device="cuda"), torch.full((N, 1), 5, dtype=torch.uint8, device="cuda")
    canon = torch.zeros(N * K // 2 + shift, dtype=torch.uint8, device="cuda")
    canon[:N * K // 2] = lib.pack_format(dev(c), lib.LAYOUT_CANONICAL, fmt).view(-1)
    Y = [torch.empty((3, N), dtype=torch.float16, device="cuda") for _ in range(2)]
    need = lib.gemm_workspace_bytes(3, N, K, 0, lib.LAYOUT_CANONICAL)
    ws = torch.empty(max(need, 256), dtype=torch.uint8, device="cuda")
    for layout, w, y in ((lib.LAYOUT_CANONICAL, canon, Y[0]), (lib.LAYOUT_TILED, dev(want), Y[1])):
        assert c_lib.w4a8_gemm_format(X.data_ptr(), sx.data_ptr(), 3, w.data_ptr(), layout, step.data_ptr(),
                                      zero.data_ptr(), N, K, 0, fmt, y.data_ptr(), 1, N, None, ws.data_ptr(),
                                      ws.numel(), None) == 0
    assert torch.equal(Y[0], Y[1])


# rows that do not fill the last set of rows of a block, a last round of columns that is partly empty, the shortest
# and longest segments of the register-resident kernel and the lengths just outside it, more than 2^21 weights in small
# groups (four rows per wave; below, and of a few rows, one; four chunks, which every four rows start elsewhere), more than 1024 and 1536 segments on both sides of the rule's lengths, every input type, rows off the vector alignment; ranges made and given
@pytest.mark.parametrize("N,K,G", [(1, 128, 128), (5, 640, 128), (6, 768, 256), (7, 1792, 256), (3, 1016, 0),
                                   (3, 1024, 0), (2, 2056, 0), (5, 9216, 0), (1, 16384, 0), (2, 16392, 0),
                                   (4, 4096, 1024), (7, 300160, 128), (5, 420608, 256), (18, 116736, 128), (21, 100096, 256),
                                   (2, 6291584, 128), (3, 4194432, 128), (21, 2048, 128), (18, 1664, 128),
                                   (1025, 1024, 0), (1537, 1536, 0), (1537, 1544, 0), (1539, 2056, 0), (513, 6144, 2048),
                                   (385, 10240, 2560)])
@pytest.mark.parametrize("dtype", ["f16", "bf16", "f32"])
def test_weight_quant_edges(lib, oracle, N, K, G, dtype):
    rng = np.random.default_rng(31 * N + K)
    pad = 8 if N % 2 else 3   # an odd stride takes the scalar loads
    W = torch.from_numpy((rng.standard_normal((N, K + pad)) * 0.02).astype(np.float32))
    W[:, K // 2] = 0.0
    W[0, :128] = 0.0                      # an empty range
    W[-1, :128] = W[-1, :128].abs()       # zero-point 0
    W = W.to({"f16": torch.float16, "bf16": torch.bfloat16, "f32": torch.float32}[dtype])
    s = rng.uniform(0.5, 2.0, K).astype(np.float32)
    Wd = W.cuda()[:, :K]
    for scale in (s, None):
        codes, step, zero = lib.quantize_weight_dint4(Wd, None if scale is None else dev(scale), G)
        rc, rs, rz = oracle.quantize_weight_dint4(W[:, :K].float().numpy(), scale, G)
        assert np.array_equal(host(step).view(np.uint32), rs.view(np.uint32))
        assert np.array_equal(host(zero), rz)
        assert np.array_equal(host(codes), rc)
    # a third of the range: most groups saturate at both ends
    st = (rs / 3).astype(np.float32)
    codes, _, _ = lib.quantize_weight_dint4(Wd, None, G, step=dev(st), zero=dev(rz))
    rc, _, _ = oracle.quantize_weight_dint4(W[:, :K].float().numpy(), None, G, step=st, zero=rz)
    assert np.array_equal(host(codes), rc)


# more rows than a grid of four per wave covers at once: the waves go on to further rows, the last of them not full
def test_weight_quant_many_rows(lib, oracle):
    N, K = 16 * 65535 + 19, 128
    g = torch.Generator(device="cuda").manual_seed(N)
    W = (torch.randn((N, K), generator=g, device="cuda", dtype=torch.float32) * 0.02).half()
    s = torch.rand((K,), generator=g, device="cuda") + 0.5
    got = lib.quantize_weight_dint4(W, s, 128)
    rows = np.r_[0:33, 16 * 65535 - 33:N]
    at = torch.from_numpy(rows).cuda()
    for a, b in zip(got, oracle.quantize_weight_dint4(host(W[at].float()), host(s), 128)):
        assert np.array_equal(host(a[at]), b)
    # the rows between, against the same rows in parts that one turn covers
    for r in range(0, N, 1 << 19):
        for a, b in zip(got, lib.quantize_weight_dint4(W[r:r + (1 << 19)], s, 128)):
            assert torch.equal(a[r:r + (1 << 19)], b)


# every tie and band edge of the rule, one binary32 step to either side of it, and values far beyond the range (within int32, where the oracle rounds): the
# steps are given, powers of two, so that u is exact
@pytest.mark.parametrize("G,K", [(128, 1024), (0, 1024), (0, 320)])
def test_code_rule_edges(lib, oracle, G, K):
    half = np.arange(-60, 61, dtype=np.float32) / 4
    u = np.concatenate([half, np.nextafter(half, np.float32(np.inf)), np.nextafter(half, np.float32(-np.inf)),
                        np.float32([-0.0, 1e9, -1e9, 63.5, -64.5, 300.0, -300.0])]).astype(np.float32)
    W = np.resize(u, (16, K)).astype(np.float32)
    ng = K // (G or K)
    zero = np.resize(np.arange(14, dtype=np.uint8), (16, ng))
    step = np.full((16, ng), 0.25, np.float32)
    rc, _, _ = oracle.quantize_weight_dint4(W * 0.25, None, G, step=step, zero=zero)
    codes, _, _ = lib.quantize_weight_dint4(dev(W * np.float32(0.25)), None, G, step=dev(step), zero=dev(zero))
    assert np.array_equal(host(codes), rc)


# Infinities and NaN: with given parameters an infinity takes the end level and NaN code 0; with ranges from the weights every
# kernel gives what the element-per-lane kernel gives on the same weights (rows off the alignment).  One and four rows per
# wave, the segment kernel, the wave-per-segment kernel.
@pytest.mark.parametrize("N,K,G", [(6, 1024, 128), (5, 420608, 256), (17, 123648, 256), (6, 2048, 0), (6, 1000, 0), (5, 512, 512)])
@pytest.mark.parametrize("dtype", ["f16", "bf16", "f32"])
def test_weight_quant_nonfinite(lib, N, K, G, dtype):
    td = {"f16": torch.float16, "bf16": torch.bfloat16, "f32": torch.float32}[dtype]
    g = torch.Generator(device="cuda").manual_seed(N + K)
    W = (torch.randn((N, K), generator=g, device="cuda") * 0.02).to(td)
    ng = K // (G or K)
    where = torch.randint(0, K, (3, N, 8), generator=g, device="cuda")
    for i, v in enumerate((float("nan"), float("inf"), -float("inf"))):
        rows = torch.arange(N, device="cuda")[i:, None] if i else torch.arange(N, device="cuda")[:, None]
        W[rows, where[i][i:] if i else where[0]] = v      # row 0: NaN only, row 1: and inf, the others: all three
    off = torch.zeros((N, K + 1), dtype=td, device="cuda")
    off[:, :K] = W
    s = torch.rand((K,), generator=g, device="cuda") + 0.5
    for scale in (s, None):
        a = lib.quantize_weight_dint4(W, scale, G)
        b = lib.quantize_weight_dint4(off[:, :K], scale, G)
        assert torch.equal(a[0], b[0]) and torch.equal(a[1].view(torch.int32), b[1].view(torch.int32)) and torch.equal(a[2], b[2])
    step = torch.full((N, ng), 0.01, device="cuda")
    zero = torch.full((N, ng), 6, dtype=torch.uint8, device="cuda")
    codes, _, _ = lib.quantize_weight_dint4(W, s, G, step=step, zero=zero)
    assert (codes[W.isnan()] == 0).all() and (codes[W == float("inf")] == 13).all() and (codes[W == -float("inf")] == 0).all()


# the same for the Value cache: the register-resident kernel, the two-sweep kernel, and rows off the alignment
@pytest.mark.parametrize("T", [1024, 512])
@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16])
def test_value_quant_nonfinite(lib, T, dtype):
    B, D = 3, 64
    g = torch.Generator(device="cuda").manual_seed(T)
    V = torch.randn((B, T, D), generator=g, device="cuda").to(dtype)
    V[0, 5, 0], V[0, 6, 1], V[1, 7, 2], V[1, 8, 3], V[1, 9, 3] = float("nan"), float("inf"), -float("inf"), float("nan"), float("inf")
    off = torch.zeros((B, T, D + 1), dtype=dtype, device="cuda")
    off[:, :, :D] = V
    a, b = lib.quantize_value_dint4(V), lib.quantize_value_dint4(off[:, :, :D])
    assert torch.equal(a[0], b[0]) and torch.equal(a[1].view(torch.int32), b[1].view(torch.int32)) and torch.equal(a[2], b[2])


# Value caches around the kernel that keeps a group in registers: the shortest and longest groups it takes and their
# neighbours, a last round of tokens that is partly empty, channels that end inside a block, heads that do not fill the
# eight XCDs, interleaved heads, rows off the alignment (general kernel)
@pytest.mark.parametrize("B,T,D,G", [(1, 896, 32, 0), (3, 384, 40, 0), (9, 1024, 64, 0), (2, 1024, 128, 0), (1, 1152, 80, 0),
                                     (5, 2048, 64, 1024), (2, 3072, 128, 1536), (1, 3072, 32, 0), (1, 4096, 128, 0), (2, 5120, 72, 0),
                                     (1, 5248, 40, 0), (2, 1040, 64, 0),
                                     # more than 6 MB of codes: one round of the group to five
                                     (49, 1024, 128, 0), (26, 2048, 128, 0), (17, 3072, 128, 1536), (18, 3072, 128, 0), (13, 4096, 128, 0),
                                     (11, 5120, 120, 0)])
@pytest.mark.parametrize("dtype,interleaved", [("f16", False), ("bf16", True), ("f16", True)])
def test_value_quant_edges(lib, oracle, B, T, D, G, dtype, interleaved):
    _, V = syn.attention_value(B + T + D, B, 1, T, D, v_dtype="f32")
    V[0, :, 0] = 0.0                      # an empty range
    V[-1, :, D - 1] = np.abs(V[-1, :, D - 1])
    td = torch.float16 if dtype == "f16" else torch.bfloat16
    if interleaved:                       # a [T, heads, D] cache
        Vd = dev(V.transpose(1, 0, 2)).to(td).transpose(0, 1)
    else:
        Vd = dev(V).to(td)
    codes, step, zero = lib.quantize_value_dint4(Vd, G)
    Vh = Vd.float().cpu().numpy()
    for b in range(B):
        rc, rs, rz = oracle.quantize_weight_dint4(np.ascontiguousarray(Vh[b].T), None, G)
        rows = slice(b * D, (b + 1) * D)
        assert np.array_equal(host(step)[rows].view(np.uint32), rs.view(np.uint32))
        assert np.array_equal(host(zero)[rows], rz)
        assert np.array_equal(host(codes)[rows], rc)


# every edge of the code rule with its two binary32 neighbours, zero-points of either parity and beyond the code space (where
# the clamp alone says what comes out): four rows and one row per wave, long segments, the wave-per-segment kernel with two and with eight columns per lane
@pytest.mark.parametrize("N,K,G", [(2050, 1024, 128), (2050, 1024, 256), (40, 256, 128), (6, 4096, 0), (3, 2304, 0), (9, 96, 48),
                                   (5, 1024, 512), (3, 768, 0)])
def test_code_rule_edges_of_kernels(lib, oracle, N, K, G):
    edges = np.concatenate([[0.0, 0.25, 0.75], np.arange(0, 31) + 0.5, np.arange(1, 31), [300.0, 2.0 ** 22]]).astype(np.float32)
    near = np.concatenate([edges, np.nextafter(edges, np.float32(np.inf)), np.nextafter(edges, np.float32(-np.inf))])
    near = np.concatenate([near, -near])
    rng = np.random.default_rng(N + K)
    W = rng.choice(near, size=(N, K)).astype(np.float32)
    ng = K // (G or K)
    zero = rng.integers(0, 14, (N, ng), dtype=np.uint8)
    zero[0], zero[1], zero[2] = 13, 200, 255
    step = np.ones((N, ng), dtype=np.float32)
    want = oracle.quantize_weight_dint4(W, None, G, step=step, zero=zero)[0]
    got = lib.quantize_weight_dint4(dev(W), None, G, step=dev(step), zero=dev(zero))[0]
    assert np.array_equal(host(got), want)


# the same edges in the Value cache's kernels (short groups, groups that stay in registers): channel d runs from -(d % 14) to
# 13 - d % 14, so that the step is 1 and the zero-point d % 14
@pytest.mark.parametrize("B,T,D,G", [(2, 256, 64, 128), (1, 1024, 48, 0), (1, 4096, 40, 0)])
@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16])
def test_value_code_rule_edges(lib, oracle, B, T, D, G, dtype):
    rng = np.random.default_rng(T + D)
    z = np.arange(D) % 14
    V = rng.integers(-4 * z[None, None, :], 4 * (13 - z)[None, None, :] + 1, (B, T, D)).astype(np.float32) / 4
    V[:, ::128], V[:, 1::128] = -z, 13 - z
    Vd = dev(V).to(dtype)
    codes, step, zero = oracle.quantize_value_dint4(host(Vd.float()), G)
    got = lib.quantize_value_dint4(Vd, G)
    assert np.array_equal(host(got[2]).reshape(zero.shape), zero) and np.array_equal(host(got[1]).reshape(step.shape), step)
    assert np.array_equal(host(got[0]).reshape(codes.shape), codes)


# every code space in the wave-per-segment kernel, whose instances differ in the special values they know: eight columns per lane
# (groups of 512, a row of 768) and two (rows off the alignment), a last round that is partly empty, with and without scales
@pytest.mark.parametrize("fmt,name,shift", [(0, "dint4", 1), (1, "int4", 1), (2, "dint3", 1), (3, "dint4", 2), (4, "dint4", 3)])
@pytest.mark.parametrize("N,K,G,pad", [(9, 1024, 512, 0), (6, 768, 0, 8), (6, 768, 0, 2)])
def test_formats_in_the_wave_per_segment_kernel(lib, oracle, fmt, name, shift, N, K, G, pad):
    rng = np.random.default_rng(N + K + fmt)
    W = (rng.standard_normal((N, K)) * 0.02).astype(np.float32).astype(np.float16)
    W[1] = np.abs(W[1])
    s = rng.uniform(0.5, 2.0, K).astype(np.float32)
    Wd = torch.zeros((N, K + pad), dtype=torch.float16, device="cuda")[:, :K]
    Wd.copy_(torch.from_numpy(W))
    for scale in (s, None):
        got = lib.quantize_weight_format(Wd, None if scale is None else dev(scale), G, fmt)
        for a, b in zip(got, oracle.formats.quantize_weight(W.astype(np.float32), scale, G, name, shift)):
            assert np.array_equal(host(a), b)
