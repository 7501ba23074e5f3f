"""Edges of the calibration kernels: token counts around the error sums' 256-token rounds and the tiles of the
unquantized product, group sizes that take the tiled quantizer and that do not, every input type."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import synthetic_inputs as syn  # noqa: E402
from gpu_util import host  # noqa: E402

pytestmark = pytest.mark.gpu
LOSS_TOL = 1e-4   # fp16 outputs against an fp32 matrix-core product: the tolerance of the search's own parity tests
DTYPES = {"f16": torch.float16, "bf16": torch.bfloat16, "f32": torch.float32}


@pytest.fixture(scope="module")
def lib():
    import paper_2311_05161_amd as w
    w.load_library()
    return w


@pytest.mark.parametrize("M,K,N,G,dtype,pad", [
    (1, 128, 16, 128, "f16", 0), (255, 256, 16, 0, "f16", 8), (257, 384, 48, 128, "f16", 0), (520, 256, 144, 256, "f16", 8),
    (3, 384, 80, 128, "bf16", 0), (129, 256, 272, 0, "bf16", 8), (70, 384, 48, 128, "bf16", 3), (65, 512, 32, 128, "f32", 4)])
def test_searches_at_edges(lib, oracle, M, K, N, G, dtype, pad):
    aq = oracle.aqas_search
    X, W, _ = syn.random_layer(M + K + N, M, K, N, x_dtype="f32", outlier_frac=0.02, outlier_gain=20.0)
    Xd, Wd = (torch.zeros((a.shape[0], K + pad), dtype=DTYPES[dtype], device="cuda") for a in (X, W))
    Xd[:, :K], Wd[:, :K] = (torch.from_numpy(a.astype(np.float32)).cuda() for a in (X, W))
    Xd, Wd = Xd[:, :K], Wd[:, :K]
    X, W = (t.float().cpu().numpy() for t in (Xd, Wd))
    ref = aq.aqas_search(X, W, G)
    s, best, losses = lib.aqas_search(Xd, Wd, G)
    losses, j = host(losses), int(host(best)[0])
    np.testing.assert_allclose(losses, ref["losses"], rtol=LOSS_TOL)
    assert losses[j] == losses.min() and np.all(losses[:j] > losses[j])
    np.testing.assert_array_equal(host(s), aq.aqas_scale(ref["ax"], ref["aw"], j))
    rc = aq.clip_search(X, W, host(s), G)
    idx, step, zero, table = lib.aqas_clip_search(Xd, Wd, s, G, want_table=True)
    idx, table = host(idx), host(table)
    # An fp16 output whose exact value lies within fp32 rounding (1e-6 relative) of a midpoint may round either way: one
    # output in some 250, i.e. at most a handful of a channel's M.  Each moves its squared difference d^2 by
    # ulp (2 |d| + ulp) at most, ulp = 2^-10 of the channel's largest output, |d| within three times its rms.
    ulp = 2.0 ** -10 * np.abs(X.astype(np.float64) @ W.astype(np.float64).T).max(axis=0) * 1.1
    bound = 6 * ulp * (6 * np.sqrt(rc["err"] / M) + ulp)
    assert np.all(np.abs(table - rc["err"]) <= 1e-5 * rc["err"] + bound)
    for n in range(N):
        assert table[idx[n], n] == table[:, n].min() and np.all(table[:idx[n], n] > table[idx[n], n])
    st, z = aq.clipped_params(W, host(s), G, np.array([aq.clip_factor(int(i)) for i in idx], np.float32))
    np.testing.assert_array_equal(host(step), st)
    np.testing.assert_array_equal(host(zero), z)


# Every channel maximum of X and W is exactly 1, so every grid point's scale is 1 and all error vectors are the same: the
# losses have to be the same bits, and the first grid point wins (the header's rule for ties).
@pytest.mark.parametrize("N", [2064, 4096, 11008])
def test_equal_scales_give_equal_losses(lib, N):
    M, K = 16, 128
    for seed in range(16):
        g = torch.Generator(device="cuda").manual_seed(seed)
        X = (torch.rand((M, K), generator=g, device="cuda") * 2 - 1).half()
        W = (torch.rand((N, K), generator=g, device="cuda") * 2 - 1).half()
        X[0], W[0] = 1.0, -1.0
        s, best, losses = lib.aqas_search(X, W, 128)
        assert (host(s) == 1.0).all()
        assert (host(losses) == host(losses)[0]).all(), (N, seed)
        assert int(host(best)[0]) == 0


# the same for candidates side by side: group-wise with one and several token tiles, a last tile of one row, per channel, all in one
# round and in several rounds of unequal size (the last two)
@pytest.mark.parametrize("M,K,N,G", [(17, 256, 2064, 128), (300, 256, 4096, 128), (257, 384, 272, 128), (300, 128, 2064, 0), (129, 512, 80, 0),
                                     (1024, 1024, 8192, 0), (1100, 1024, 12288, 128)])
def test_equal_scales_give_equal_losses_side_by_side(lib, M, K, N, G):
    c = lib.load_library()
    assert c.aqas_search_workspace_preferred_bytes(M, N, K, G) > c.aqas_search_workspace_bytes(M, N, K, G) + 3 * M * K
    for seed in range(4):
        g = torch.Generator(device="cuda").manual_seed(seed)
        X = (torch.rand((M, K), generator=g, device="cuda") * 2 - 1).half()
        W = (torch.rand((N, K), generator=g, device="cuda") * 2 - 1).half()
        X[0], W[0] = 1.0, -1.0
        s, best, losses = lib.aqas_search(X, W, G)
        assert (host(s) == 1.0).all()
        assert (host(losses) == host(losses)[0]).all(), seed
        assert int(host(best)[0]) == 0


# A workspace of the size that one candidate at a time needs is enough, whatever the search would like to have; candidates
# side by side (several rounds of them on the last shape) see the same errors to fp16 rounding of single outputs.
@pytest.mark.parametrize("M,K,N,G,dtype", [(17, 128, 16, 128, "f16"), (300, 384, 272, 128, "bf16"), (64, 8192, 64, 128, "f16"),
                                           (129, 512, 80, 0, "f32"), (1100, 1024, 12288, 128, "f16")])
def test_side_by_side_against_one_by_one(lib, M, K, N, G, dtype):
    g = torch.Generator(device="cuda").manual_seed(M)
    X = torch.randn((M, K), generator=g, device="cuda")
    X[:, :: 37] *= 20.0
    X, W = X.to(DTYPES[dtype]), (torch.randn((N, K), generator=g, device="cuda") * 0.02).to(DTYPES[dtype])
    c, i32, f64 = lib.load_library(), torch.int32, torch.float64
    code = {"f32": 0, "f16": 1, "bf16": 2}[dtype]
    full, small = int(c.aqas_search_workspace_preferred_bytes(M, N, K, G)), int(c.aqas_search_workspace_bytes(M, N, K, G))
    # what one candidate at a time needs, from its parts; side by side needs more (the operands of 17 candidates, or of fewer in
    # several rounds), so that the two sizes are two paths
    part = [3 * 4 * K, M * K, 4 * M, N * K, 5 * N * (K // (G or K)), N * K // 2, 6 * M * N, 16 * N,
            int(c.w4a8_gemm_workspace_bytes(M, N, K, G, 1))]
    assert sum(part) <= small <= sum(part) + 256 * 16 and small + 3 * M * K < full
    out = {}
    for need in (full, small):
        ws = torch.full((need,), 255, dtype=torch.uint8, device="cuda")
        s, best, losses = (torch.empty(n, dtype=t, device="cuda") for n, t in ((K, torch.float32), (1, i32), (17, f64)))
        stream = torch.cuda.current_stream().cuda_stream
        assert c.aqas_search(X.data_ptr(), W.data_ptr(), code, M, N, K, K, K, G, s.data_ptr(), best.data_ptr(),
                             losses.data_ptr(), ws.data_ptr(), need, stream) == 0
        ng = K // (G or K)
        idx, step, zero, table = (torch.empty(n, dtype=t, device="cuda") for n, t in
                                  ((N, i32), (N * ng, torch.float32), (N * ng, torch.uint8), (11 * N, f64)))
        j = int(host(best)[0])
        s.fill_(1.25)
        assert c.aqas_clip_search(X.data_ptr(), W.data_ptr(), code, M, N, K, K, K, s.data_ptr(), G, idx.data_ptr(),
                                  step.data_ptr(), zero.data_ptr(), table.data_ptr(), ws.data_ptr(), need, stream) == 0
        out[need] = (host(losses), host(table).reshape(11, N), j, host(idx), host(step), host(zero))
    np.testing.assert_allclose(out[full][0], out[small][0], rtol=LOSS_TOL)
    # single channels: a few outputs may round the other way, each by one fp16 step of its value (see the bound above)
    ulp = 2.0 ** -10 * host((X.float() @ W.float().t()).abs().amax(0)).astype(np.float64) * 1.1
    err = out[small][1]
    bound = 6 * ulp * (6 * np.sqrt(err / M) + ulp)
    assert np.all(np.abs(out[full][1] - err) <= 1e-5 * err + bound)
    # the same winners, but for grid points and factors whose errors are equal to within that
    j, k = out[full][2], out[small][2]
    assert out[small][0][j] <= out[small][0][k] * (1 + 2 * LOSS_TOL)
    a, b = out[full][3], out[small][3]
    n = np.arange(N)
    gap = err[a, n] - err[b, n]
    assert np.all((gap >= 0) & (gap <= 2e-5 * err[a, n] + bound[a, n] + bound[b, n]))
    same = a == b
    print(f"grid point {j} / {k}, clipping factors the same in {same.mean():.4f} of {N} channels")
    ng = K // (G or K)
    for p in (4, 5):
        np.testing.assert_array_equal(out[full][p].reshape(N, ng)[same], out[small][p].reshape(N, ng)[same])


# rows further apart than a buffer descriptor reaches (2^26 elements), in X, in W and in both: the same bits as dense rows
@pytest.mark.parametrize("far_x,far_w", [(True, False), (False, True), (True, True)])
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_rows_far_apart(lib, far_x, far_w, dtype):
    M, K, N, stride = 70, 384, 48, (1 << 26) + 8
    g = torch.Generator(device="cuda").manual_seed(7)
    dense = [(torch.randn((rows, K), generator=g, device="cuda") * scale).to(DTYPES[dtype]) for rows, scale in ((M, 1.0), (N, 0.02))]
    spread = []
    for t, far in zip(dense, (far_x, far_w)):
        if far:
            wide = torch.empty((t.shape[0], stride), dtype=t.dtype, device="cuda")[:, :K]
            wide.copy_(t)
            t = wide
        spread.append(t)
    assert spread[0].stride(0) == (stride if far_x else K) and spread[1].stride(0) == (stride if far_w else K)
    want, got = (lib.aqas_search(X, W, 128) for X, W in (dense, spread))
    assert all(torch.equal(a, b) for a, b in zip(want, got))
    want, got = (lib.aqas_clip_search(X, W, want[0], 128, want_table=True) for X, W in (dense, spread))
    assert all(torch.equal(a, b) for a, b in zip(want, got))


# The quantizers that write packed weights (one candidate at a time) and int8 weights (side by side), at the edges of the code rule with
# both neighbours: every group runs from -z to 13 - z, so that its step is 1, and token m excites channel m and one whose weight
# lies 0.3 off its level, so that the two sides of a tie differ in the squared error -- by 0.3 * 127^2 for one code, 1e-3 of a
# row's sum, against 4e-5 for the rounding of the binary32 product (1e-4 of 6 in a difference, squared).
@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("side_by_side", [False, True])
def test_clipping_errors_at_the_rule_edges(lib, oracle, dtype, side_by_side):
    M, K, N, G = 256, 256, 32, 128
    rng = np.random.default_rng(3)
    W = np.empty((N, K), np.float32)
    for n in range(N):
        z = n % 14
        half = np.concatenate([np.arange(-z, 13 - z) + 0.5, [-0.75, -0.25, 0.25, 0.75]])
        half = torch.from_numpy(half[(half > -z) & (half < 13 - z)]).to(DTYPES[dtype])
        inf = torch.tensor(float("inf"), dtype=half.dtype)
        edges = torch.cat([half, torch.nextafter(half, inf), torch.nextafter(half, -inf)]).float().numpy()
        W[n] = np.concatenate([rng.permutation(np.resize(rng.permutation(edges), G)) for _ in range(K // G)])
        W[n, 0::G], W[n, 1::G], W[n, 2::G] = -z, 13 - z, 1.296875 if z < 11 else -1.296875   # (exact in every type)
    X = np.zeros((M, K), np.float32)
    X[np.arange(M), np.arange(M)] = X[np.arange(M), np.arange(M) // G * G + 2] = 127.0
    s = np.ones(K, np.float32)
    want = oracle.aqas_search.clip_search(X, W, s, G)["err"][0]
    Xd, Wd, sd = (torch.from_numpy(a).cuda() for a in (X, W, s))
    Xd, Wd = Xd.to(DTYPES[dtype]), Wd.to(DTYPES[dtype])
    c = lib.load_library()
    full, small = int(c.aqas_search_workspace_preferred_bytes(M, N, K, G)), int(c.aqas_search_workspace_bytes(M, N, K, G))
    assert full > small + 10 * N * K
    need = full if side_by_side else small
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    idx, step, zero, table = (torch.empty(n, dtype=t, device="cuda") for n, t in
                              ((N, torch.int32), (N * K // G, torch.float32), (N * K // G, torch.uint8), (11 * N, torch.float64)))
    assert c.aqas_clip_search(Xd.data_ptr(), Wd.data_ptr(), {"f32": 0, "f16": 1, "bf16": 2}[dtype], M, N, K, K, K, sd.data_ptr(), G,
                              idx.data_ptr(), step.data_ptr(), zero.data_ptr(), table.data_ptr(), ws.data_ptr(), need,
                              torch.cuda.current_stream().cuda_stream) == 0
    np.testing.assert_allclose(host(table).reshape(11, N)[0], want, rtol=1e-4)
