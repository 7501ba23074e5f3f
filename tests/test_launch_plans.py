"""The rules that choose a launch, read from the built library on the CPU (nothing is launched)."""
import ctypes

import pytest

import paper_2311_05161_amd as w

I64 = ctypes.c_int64


class GemvPlan(ctypes.Structure):   # csrc/w4a8_common.hpp
    _fields_ = [(n, ctypes.c_int) for n in ("splits", "kt_per_split", "at", "q", "blocks_per_split", "nt_lo", "nt_rem",
                                            "lds_bytes")] + [("partial_bytes", ctypes.c_size_t)]


class GemmPlan(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int) for n in ("bm", "splits", "kt_per_split")] + [
        (n, ctypes.c_size_t) for n in ("rs_bytes", "partial_bytes")] + [
        (n, ctypes.c_int) for n in ("rem_n", "rem_splits", "rem_kt_per_split", "pc_rem_n")]


class MidForm(ctypes.Structure):
    _fields_ = [("phases", ctypes.c_int), ("blocks", ctypes.c_int)]


def _rule(symbol, restype, *argtypes):
    f = w.load_library()["_ZN4w4a8" + symbol]
    f.restype, f.argtypes = restype, argtypes
    return f


def plan_gemv(M, N, K, G, batch=1, token_blocks=False):
    f = _rule("9plan_gemvElllllb", GemvPlan, I64, I64, I64, I64, I64, ctypes.c_bool)
    return f(M, N, K, G or K, batch, token_blocks)


def route(M, K, N, G, asym=False):
    """The kernel that a product of more than 16 tokens runs on: ("phases", phases, token blocks), ("stream", blocks),
    ("phases per channel",) or ("tile", rows, K ranges, channels of the last round that run with K in ranges)."""
    G = G or K
    r = _rule("13gemm_mid_formEllllb", MidForm, I64, I64, I64, I64, ctypes.c_bool)(M, N, K, G, asym)
    if r.phases:
        return "phases", r.phases, r.blocks
    blocks = _rule("17gemv_token_blocksEllll", ctypes.c_int, I64, I64, I64, I64)(M, N, K, G)
    if blocks:
        return "stream", blocks
    if _rule("19gemm_mid_pc_appliesEllllb", ctypes.c_bool, I64, I64, I64, I64, ctypes.c_bool)(M, N, K, G, asym):
        return ("phases per channel",)
    p = _rule("9plan_gemmEllll", GemmPlan, I64, I64, I64, I64)(M, N, K, G)
    return "tile", p.bm, p.splits, p.rem_n


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


def mid_phases(M, N, K, asym):
    return _rule("15gemm_mid_phasesEllllb", ctypes.c_int, I64, I64, I64, I64, ctypes.c_bool)(M, N, K, 128, asym)


# group-128 weights, one shape on either side of each line at which the four-block form of the K-phase kernel and the tile kernel
# were timed against each other (the times stand beside the rule).  Where these lines say yes, the cost rule (gemm_mid_form, which
# decides) compares the other forms with this one and not with the tile kernel.
@pytest.mark.parametrize("M,K,N,asym,phases", [
    (512, 5120, 2560, False, 4), (256, 8192, 5120, False, 4), (230, 6144, 3200, False, 4), (192, 12800, 5760, False, 4),
    (250, 9728, 4608, False, 4), (256, 13824, 5120, False, 4), (150, 1536, 1552, False, 4), (129, 1280, 1168, False, 4), (230, 3584, 1984, False, 0),
    (230, 11008, 3840, False, 0), (140, 8192, 3840, False, 0), (450, 7168, 1344, False, 0), (135, 2176, 1152, False, 0),
    (230, 6144, 3840, True, 4), (640, 5120, 1792, True, 4), (384, 8192, 2560, True, 0), (512, 4096, 768, True, 0),
    (256, 2048, 2048, True, 0), (1024, 4096, 4096, False, 2), (512, 13824, 5120, False, 0), (1024, 1024, 4096, False, 0)])
def test_four_block_lines(M, K, N, asym, phases):
    assert mid_phases(M, N, K, asym) == phases


# per-channel layers a few tiles beyond whole rounds: the channels that go to the K-phase kernel, none below K = 3072
@pytest.mark.parametrize("M,K,N,rem_n", [
    (1531, 4096, 11008, 256), (1100, 3072, 14480, 144), (1100, 3200, 14592, 256), (3495, 3072, 4656, 48), (700, 9216, 22016, 256),
    (1100, 1024, 14480, 0), (1934, 2048, 8672, 0), (2394, 2560, 6832, 0), (1100, 9344, 14480, 0), (4140, 3072, 4112, 0),
    (2048, 4096, 8192, 0)])
def test_per_channel_remainder(M, K, N, rem_n):
    pl = _rule("9plan_gemmEllll", GemmPlan, I64, I64, I64, I64)(M, N, K, K)
    assert pl.pc_rem_n == rem_n and pl.splits == 1


# what decides, at the shapes of the edge tests: every one but a token-block shape and the last three is on the K-phase kernel
def test_edge_shapes_take_their_kernels():
    from test_gpu_mid_edges import FOUR, TILE, TWO
    for asym in (False, True):
        got = [route(*s, 128, asym) for s in FOUR + TWO + TILE]
        assert got[0] == ("stream", 5) and [r[0] for r in got[1:-3]] == ["phases"] * (len(got) - 4)
        assert got[-3:] == [("tile", 128, 1, 0)] * 3
