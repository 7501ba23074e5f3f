"""The natively marshalled calls against the binding's Python forms: same outputs, same refusals."""
import ctypes
import threading

import numpy as np
import pytest

torch = pytest.importorskip("torch")

import paper_2311_05161_amd as w  # noqa: E402
from paper_2311_05161_amd import binding  # noqa: E402

pytestmark = pytest.mark.gpu


class Sub(torch.Tensor):
    pass


def _layer(M, K, N, G, dtype=torch.float16, pad=0):
    g = torch.Generator(device="cuda").manual_seed(M + K + N)
    X = torch.randn((M, K + pad), generator=g, device="cuda").to(dtype)[:, :K]
    s = torch.rand((K,), generator=g, device="cuda") + 0.5
    W = torch.randn((N, K), generator=g, device="cuda").half() * 0.02
    codes, step, zero = w.quantize_weight_dint4(W, s, G)
    return X, s, w.pack_dint4(codes), step, zero, w.dint4_weight_sums(codes, zero, G)


# one launch, two launches (bfloat16, K in ranges, strided rows off the alignment), a workspace, no tokens
@pytest.mark.parametrize("M,K,N,G,dtype,pad", [
    (1, 512, 256, 128, torch.float16, 0), (16, 5120, 48, 0, torch.bfloat16, 8), (5, 11008, 32, 0, torch.float16, 0),
    (3, 512, 64, 128, torch.float32, 1), (200, 1024, 272, 0, torch.float16, 0), (0, 256, 32, 128, torch.float16, 0)])
def test_native_forms_equal_python_forms(M, K, N, G, dtype, pad):
    X, s, Wp, step, zero, (wsum, tsum) = _layer(M, K, N, G, dtype, pad)
    for scale in (s, None):
        Xq, sx = w.quantize_act_int8(X, scale)
        Xq2, sx2 = w.quantize_act_int8(X, scale, Xq=torch.empty_like(Xq))
        assert torch.equal(Xq, Xq2) and torch.equal(sx, sx2)
        Aq, ax, az = w.quantize_act_int8_asym(X, scale)
        Aq2, ax2, az2 = w.quantize_act_int8_asym(X, scale, zx=torch.empty_like(az))
        assert torch.equal(Aq, Aq2) and torch.equal(ax, ax2) and torch.equal(az, az2)
        for yd in (torch.float16, torch.bfloat16):
            def fresh():
                return torch.empty((M, N), dtype=yd, device="cuda")
            Y = w.w4a8_linear(X, scale, Wp, step, zero, N, G, out_dtype=yd)
            assert Y.dtype == yd and torch.equal(Y, w.w4a8_linear(X, scale, Wp, step, zero, N, G, Y=fresh()))
            Y = w.w4a8_gemm(Xq, sx, Wp, step, zero, N, K, G, out_dtype=yd)
            assert torch.equal(Y, w.w4a8_gemm(Xq, sx, Wp, step, zero, N, K, G, Y=fresh()))
            Y = w.w4a8_gemm_asym(Aq, ax, az, Wp, step, zero, wsum, tsum, N, K, G, out_dtype=yd)
            assert torch.equal(Y, w.w4a8_gemm_asym(Aq, ax, az, Wp, step, zero, wsum, tsum, N, K, G, Y=fresh()))


def test_refusals_and_forms_left_to_python():
    X, s, Wp, step, zero, _ = _layer(4, 512, 64, 128)
    ref = w.w4a8_linear(X, s, Wp, step, zero, 64, 128)
    assert torch.equal(w.w4a8_linear(X.as_subclass(Sub), s, Wp, step, zero, 64, 128), ref)
    for bad, status in ((dict(N=60), binding.ERR_SHAPE), (dict(group_size=100), binding.ERR_SHAPE),
                        (dict(layout=7), binding.ERR_DTYPE), (dict(out_dtype=torch.float32), binding.ERR_DTYPE)):
        with pytest.raises(w.W4A8Error) as e:
            w.w4a8_linear(X, s, Wp, step, zero, **{**dict(N=64, group_size=128), **bad})
        assert e.value.status == status
    with pytest.raises(ValueError):
        w.quantize_act_int8(X.t())
    with pytest.raises(KeyError):
        w.quantize_act_int8(X.to(torch.int32))
    with pytest.raises(KeyError):
        w.w4a8_linear(X, s, Wp, step, zero, 64, 128, out_dtype=torch.int32)


# a card that has room for the scratch that a call has to have but not for what it would like: the same bits as with room
@pytest.mark.parametrize("native", [True, False])
def test_scratch_that_cannot_be_had(native, monkeypatch):
    M, K, N, G = 2048, 5120, 13824, 128
    X, s, Wp, step, zero, _ = _layer(M, K, N, G)
    Xq, sx = w.quantize_act_int8(X, s)
    Wc, Xc = torch.randn((2048, 2048), device="cuda").half(), torch.randn((512, 2048), device="cuda").half()
    if not native:
        monkeypatch.setattr(binding, "_native", False)
    lib = w.load_library()
    calls = [(lambda: w.w4a8_gemm(Xq, sx, Wp, step, zero, N, K, G), w.gemm_workspace_bytes(M, N, K, G),
              w.gemm_workspace_preferred_bytes(M, N, K, G), 2 * M * N),
             (lambda: w.w4a8_linear(X, s, Wp, step, zero, N, G), w.linear_workspace_bytes(M, N, K, G),
              w.linear_workspace_preferred_bytes(M, N, K, G), 2 * M * N),
             (lambda: w.aqas_clip_search(Xc, Wc, torch.ones(2048, device="cuda"), G)[1],
              lib.aqas_search_workspace_bytes(512, 2048, 2048, G), lib.aqas_search_workspace_preferred_bytes(512, 2048, 2048, G), 1 << 21)]
    total = torch.cuda.mem_get_info()[1]
    for call, least, preferred, out in calls:
        ref = call()
        assert preferred > least + (48 << 20)
        torch.cuda.empty_cache()
        held, reserved = [], torch.cuda.memory_reserved()
        try:
            torch.cuda.set_per_process_memory_fraction(reserved / total)
            for size in (64 << 20, 8 << 20, 2 << 20):      # what is free inside the allocator's blocks
                with pytest.raises(torch.OutOfMemoryError):
                    while True:
                        held.append(torch.empty((size,), dtype=torch.uint8, device="cuda"))
            torch.cuda.set_per_process_memory_fraction((reserved + least + out + (24 << 20)) / total)   # (it grows by 2 to 20 MB at a time)
            with pytest.raises(torch.OutOfMemoryError):
                [torch.empty((n,), dtype=torch.uint8, device="cuda") for n in (out, preferred)]
            torch.cuda.empty_cache()
            got = call()
        finally:
            torch.cuda.set_per_process_memory_fraction(1.0)
        if ref.dtype == torch.float32:   # (steps; a factor may flip where two have the same error)
            assert float((got != ref).float().mean()) < 1e-2
        else:
            assert torch.equal(got, ref)


def test_current_stream_and_threads():
    X, s, Wp, step, zero, _ = _layer(16, 4096, 512, 128)
    ref = w.w4a8_linear(X, s, Wp, step, zero, 512, 128)
    bad = []

    def work():
        st = torch.cuda.Stream()
        st.wait_stream(torch.cuda.default_stream())
        with torch.cuda.stream(st):
            for _ in range(50):
                Xi = X.clone()      # made on this stream just before
                if not torch.equal(w.w4a8_linear(Xi, s, Wp, step, zero, 512, 128), ref):
                    bad.append(1)

    torch.cuda.synchronize()
    threads = [threading.Thread(target=work) for _ in range(4)]
    [t.start() for t in threads]
    [t.join() for t in threads]
    assert not bad
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        Y = w.w4a8_linear(X, s, Wp, step, zero, 512, 128)
        Z = w.w4a8_linear(X.float(), s, Wp, step, zero, 512, 128)     # two launches, a workspace
    for _ in range(3):
        Y.zero_(), Z.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(Y, ref) and torch.equal(Z, ref)


# what the Python forms convert stays accepted, what they refuse stays refused, with and without a given output
def test_sizes_that_are_not_ints():
    M, K, N = 4, 512, 64
    X, s, Wp, step, zero, (wsum, tsum) = _layer(M, K, N, 128)
    Xq, sx = w.quantize_act_int8(X, s)
    Aq, ax, az = w.quantize_act_int8_asym(X, s)

    def calls(n=N, **kw):
        for Y in (None, torch.empty((M, N), dtype=torch.float16, device="cuda")):
            yield lambda: w.w4a8_linear(X, s, Wp, step, zero, n, Y=Y, **kw)
            yield lambda: w.w4a8_gemm(Xq, sx, Wp, step, zero, n, K, Y=Y, **kw)
            yield lambda: w.w4a8_gemm_asym(Aq, ax, az, Wp, step, zero, wsum, tsum, n, K, Y=Y, **kw)

    ref = [f().clone() for f in calls(group_size=128)]
    for kw in (dict(group_size=128.0), dict(group_size="128"), dict(group_size=np.int64(128)),
               dict(group_size=128, layout=float(w.LAYOUT_TILED)), dict(group_size=128, layout=str(w.LAYOUT_TILED))):
        for f, r in zip(calls(**kw), ref):
            assert torch.equal(f(), r)
    for f, r in zip(calls(n=np.int64(N), group_size=128), ref):
        assert torch.equal(f(), r)
    for f in calls(n=float(N), group_size=128):
        with pytest.raises((ctypes.ArgumentError, TypeError)):
            f()


# an output or workspace that does not fit raises what torch.empty raises (callers catch it to shrink a batch)
def test_out_of_memory_is_torch_s_own():
    X, s, Wp, step, zero, (wsum, tsum) = _layer(4096, 512, 64, 128)
    Xq, sx = w.quantize_act_int8(X, s)
    Aq, ax, az = w.quantize_act_int8_asym(X, s)
    # 8 GiB of outputs where the allocator may hold 1 % of the card; a call that got past it would be refused
    # for its group size before any launch
    N, G = 1 << 20, 100
    torch.cuda.empty_cache()
    torch.cuda.set_per_process_memory_fraction(0.01)
    try:
        for f in (lambda: w.w4a8_linear(X, s, Wp, step, zero, N, G),
                  lambda: w.w4a8_gemm(Xq, sx, Wp, step, zero, N, 512, G),
                  lambda: w.w4a8_gemm_asym(Aq, ax, az, Wp, step, zero, wsum, tsum, N, 512, G)):
            with pytest.raises(torch.OutOfMemoryError):
                f()
    finally:
        torch.cuda.set_per_process_memory_fraction(1.0)
    assert w.w4a8_linear(X, s, Wp, step, zero, 64, 128).shape == (4096, 64)


# without the extension every call takes its Python form
def test_calls_without_the_extension(monkeypatch):
    X, s, Wp, step, zero, (wsum, tsum) = _layer(5, 1024, 64, 128)

    def calls():
        Xq, sx = w.quantize_act_int8(X, s)
        Aq, ax, az = w.quantize_act_int8_asym(X, s)
        return (Xq, sx, Aq, ax, az, w.w4a8_linear(X, s, Wp, step, zero, 64, 128),
                w.w4a8_gemm(Xq, sx, Wp, step, zero, 64, 1024, 128),
                w.w4a8_gemm_asym(Aq, ax, az, Wp, step, zero, wsum, tsum, 64, 1024, 128))

    ref = calls()
    monkeypatch.setattr(binding, "_native", False)
    assert all(torch.equal(a, b) for a, b in zip(calls(), ref))
