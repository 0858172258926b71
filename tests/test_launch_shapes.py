"""Host-side rules that shape launches: column tiles and rows per tile of the full-width
matrix product, and which layers run as one kernel.  No GPU: the rules take the card's sizes as arguments."""
import ctypes

import pytest

from paper_2401_06145_amd import binding as B

CUS = 256


class _Seg(ctypes.Structure):
    _fields_ = [("k", ctypes.c_int), ("row0", ctypes.c_int64), ("rows", ctypes.c_int64), ("height", ctypes.c_int64)]


def _wide_tiles(heights, c_in, c_out, elem, per_cu=1):
    segs, at = (_Seg * len(heights))(), 0
    for i, h in enumerate(heights):
        segs[i] = _Seg(i, at, h, h)
        at += h
    nt, rows = ctypes.c_int(), ctypes.c_int()
    i64, c_int = ctypes.c_int64, ctypes.c_int
    # void spc::wide_tiles(const GemmSeg*, int, int, int, int, int64_t, int64_t, int*, int*)
    B.lib()._ZN3spc10wide_tilesEPKNS_7GemmSegEiiiillPiS3_(
        segs, c_int(len(heights)), c_int(c_in), c_int(c_out), c_int(elem), i64(CUS), i64(per_cu), ctypes.byref(nt),
        ctypes.byref(rows))
    return nt.value, rows.value, sum(-(-h // rows.value) for h in heights) * (c_out // 16 // nt.value)


@pytest.mark.parametrize("heights,c_in,c_out,nt,rows", [
    ([4096] * 8, 384, 256, 8, 512),           # K = 2 stride 2, two slices: 128 workgroups
    ([32768], 512, 192, 6, 512),              # K = 1, two slices: 128 workgroups
    ([512] * 128, 160, 64, 4, 512),           # one slice
    ([512] * 128, 64, 64, 2, 128),            # the same with fewer weights: half slices
    ([2000] + [15] * 124, 384, 128, 4, 128),  # 128 workgroups, most of few rows
])
def test_exactly_half_the_card(heights, c_in, c_out, nt, rows):
    """Exactly half the CUs with a workgroup: long tiles with many weights stay at 512 rows
    and the full slice, others take half slices."""
    assert _wide_tiles(heights, c_in, c_out, 2)[:2] == (nt, rows)


def test_fewer_workgroups_shrink_tiles_then_slices():
    nt, rows, wg = _wide_tiles([500] * 127, 64, 128, 2)     # one short of half
    assert (nt, rows) == (8, 256) and wg >= CUS // 2
    nt, rows, wg = _wide_tiles([600], 256, 256, 2)
    assert (nt, rows) == (1, 128) and wg == 5 * 16


@pytest.mark.parametrize("heights,c_in,c_out,rows", [
    ([2000] + [15] * 26, 128, 512, 128),      # scattered voxels: one long segment
    ([8001] + [60] * 63, 256, 128, 128),
    ([3000] * 8, 64, 64, 128),                # 94 rows for each CU
    ([20000] * 4, 64, 64, 384),               # 312 rows for each CU
    ([20000] * 4, 64, 512, 512),
    ([120000] + [8000] * 26, 64, 64, 768),    # 641 rows for each of two rounds of tiles: two row blocks
    ([120000] + [8000] * 26, 128, 64, 768),   # (one)
    ([200000] + [8000] * 26, 64, 64, 1024),   # 797 rows
    ([200000] + [8000] * 26, 128, 64, 896),
])
def test_float32_tiles_follow_the_work(heights, c_in, c_out, rows):
    """float32 tiles hold one CU's share of the rows times column slices, 128 to 512 rows
    (whole rounds of 128; of 256 from 512 rows at 33 to 64 channels, where a wave takes two row
    blocks), before the rule for large launches."""
    assert _wide_tiles(heights, c_in, c_out, 4)[1] == rows


@pytest.mark.parametrize("c_in,dtype,rows,general", [
    (4, "F32", 2 ** 18 - 1, True), (4, "F32", 2 ** 18, False), (8, "F32", 1, True), (8, "F32", 10 ** 6, False),
    (12, "F32", 1, False), (256, "F32", 1, False), (8, "F16", 1, False), (8, "BF16", 1, False),
])
def test_narrowest_float32_inputs_take_the_general_product(c_in, dtype, rows, general):
    """Less than a k-step of the full-width product, unless there are many rows."""
    f = B.lib()._ZN3spc12gemm_generalEiil
    f.restype = ctypes.c_bool
    assert f(c_in, getattr(B, "SPCONV_" + dtype), ctypes.c_int64(rows)) == general


F32, F16, BF16 = B.SPCONV_F32, B.SPCONV_F16, B.SPCONV_BF16


@pytest.mark.parametrize("n_out,per_out,K,c_in,c_out,dtype,one", [
    (60_000, 2.9, 3, 32, 64, F16, True),        # 108 KiB of weights
    (60_000, 2.9, 3, 48, 48, F16, False),       # 162 KiB
    (60_000, 2.9, 3, 64, 32, BF16, True),
    (60_000, 2.9, 3, 64, 48, F16, False),
    (60_000, 6.8, 5, 8, 64, F16, True),
    (60_000, 6.8, 5, 8, 96, F16, False),
    (60_000, 1.0, 2, 96, 96, F16, True),
    (60_000, 2.9, 3, 64, 16, F16, True),        # two k-steps, one tile
    (60_000, 2.9, 3, 96, 16, F16, False),       # three
    (60_000, 1.0, 1, 128, 32, F16, False),      # one launch in separate steps as well
    (60_000, 1.0, 1, 64, 16, F16, True),        # (not with one tile)
    (60_000, 1.0, 1, 96, 32, F16, True),
    (8191, 2.9, 3, 32, 64, F16, False),         # few outputs, 108 KiB
    (8192, 2.9, 3, 32, 64, F16, True),
    (8191, 3.3, 3, 32, 64, F16, True),
    (500, 1.1, 3, 32, 32, F16, True),           # 54 KiB
    (500, 1.0, 2, 64, 64, F16, True),           # 64 KiB
    (500, 1.0, 2, 64, 96, F16, False),
    (500, 1.0, 2, 64, 96, BF16, False),
    (60_000, 2.9, 3, 16, 64, F32, True),
    (60_000, 2.9, 3, 16, 96, F32, False),       # more than four k-steps x tiles
    (60_000, 1.1, 3, 16, 64, F32, False),       # hardly any neighbours
    (60_000, 2.9, 3, 32, 32, F32, False),       # two k-steps, sparse
    (60_000, 3.3, 3, 32, 32, F32, True),
    (500, 1.9, 5, 32, 16, F16, True),           # 125 offsets of few pairs
    (500, 1.9, 5, 8, 32, F32, True),
    (60_000, 1.2, 3, 16, 64, F32, True),
    (60_000, 1.0, 2, 32, 32, F32, True),
    (60_000, 1.0, 1, 64, 128, F32, True),
    (2000, 1.1, 3, 16, 16, F32, True),
    (2000, 1.1, 3, 16, 32, F32, False),         # few outputs, two tiles
    (2000, 1.1, 3, 8, 32, F32, False),
    (2000, 1.1, 3, 4, 32, F32, True),           # four offsets per step
    (2000, 7.4, 3, 16, 32, F32, True),
    (2000, 7.4, 3, 16, 48, F32, False),
])
def test_layers_that_run_as_one_kernel(n_out, per_out, K, c_in, c_out, dtype, one):
    assert _one_kernel(n_out, n_out, int(n_out * per_out), K, c_in, c_out, dtype) == one


def test_one_kernel_positions_stay_in_32_bits():
    """A transposed K = 1 map may have close to 2^31 outputs; positions past the last output
    that the kernel looks ahead to must not wrap."""
    assert _one_kernel(1000, 2 ** 31 - 2 ** 17, 1000, 1, 16, 16, F16)
    assert not _one_kernel(1000, 2 ** 31 - 2 ** 15, 1000, 1, 16, 16, F16)
    # input rows are addressed in 32 bits below the offset that stands for none
    assert _one_kernel(7 * 2 ** 26, 1000, 1000, 1, 8, 16, F32) is False
    assert _one_kernel(7 * 2 ** 24, 1000, 1000, 1, 8, 16, F32)


def _one_kernel(n_in, n_out, pairs, K, c_in, c_out, dtype):
    i64, c_int = ctypes.c_int64, ctypes.c_int
    # bool spc::conv_small_applies(int64_t, int64_t, int64_t, int, int, int, int)
    f = B.lib()._ZN3spc18conv_small_appliesEllliiii
    f.restype = ctypes.c_bool
    return f(i64(n_in), i64(n_out), i64(pairs), c_int(K ** 3), c_int(c_in), c_int(c_out), c_int(dtype))
