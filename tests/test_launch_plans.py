"""The rules that choose a launch, read from the built library on the CPU (nothing is launched)."""
import ctypes

import pytest

import paper_2311_05161_amd as w

I64 = ctypes.c_int64


class GemvPlan(ctypes.Structure):   # csrc/w4a8_common.hpp
    _fields_ = [(n, ctypes.c_int) for n in ("splits", "kt_per_split", "at", "q", "blocks_per_split", "nt_lo", "nt_rem",
                                            "lds_bytes")] + [("partial_bytes", ctypes.c_size_t)]


def _rule(symbol, restype, *argtypes):
    f = w.load_library()["_ZN4w4a8" + symbol]
    f.restype, f.argtypes = restype, argtypes
    return f


def plan_gemv(M, N, K, G, batch=1, token_blocks=False):
    f = _rule("9plan_gemvElllllb", GemvPlan, I64, I64, I64, I64, I64, ctypes.c_bool)
    return f(M, N, K, G or K, batch, token_blocks)


# problems with weights of their own: all the workgroups that fit 256 CUs; 16-token blocks of one problem: a multiple of
# eight per block where no workgroup gets more n-tiles for it
@pytest.mark.parametrize("batch,M,N,K,G", [(7, 1, 4096, 4096, 0), (12, 16, 1024, 1024, 0), (3, 1, 4096, 4096, 128),
                                           (20, 1, 208, 4096, 0)])
def test_batched_problems_keep_their_workgroups(batch, M, N, K, G):
    pl = plan_gemv(M, N, K, G, batch)
    assert pl.splits == 1 and pl.blocks_per_split == min(256 // batch, N // 16)
    assert pl.nt_lo * pl.blocks_per_split + pl.nt_rem == N // 16
    blocks = plan_gemv(16, N, K, G, batch, True)
    assert blocks.q == pl.q and blocks.blocks_per_split <= pl.blocks_per_split


def test_token_blocks_are_rounded_to_eight():
    for N, K, G in ((4096, 4096, 128), (5120, 5120, 0), (11008, 4096, 128)):
        pl = plan_gemv(16, N, K, G, 3, True)
        assert pl.blocks_per_split * pl.splits % 8 == 0
