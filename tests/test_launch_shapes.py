"""Host-side rules that shape launches: column tiles and rows per tile of the full-width
matrix product.  No GPU: the rules take the card's sizes as arguments."""
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
    ([4096] * 8, 384, 256, 8, 512),     # K = 2 stride 2, two slices: 128 workgroups
    ([32768], 512, 192, 6, 512),        # K = 1, two slices: 128 workgroups
    ([512] * 128, 32, 64, 4, 512),      # one slice
])
def test_half_the_card_keeps_its_tiles(heights, c_in, c_out, nt, rows):
    """Exactly half the CUs with a workgroup: tiles stay at 512 rows and the full slice."""
    assert _wide_tiles(heights, c_in, c_out, 2) == (nt, rows, CUS // 2)


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
    ([120000] + [8000] * 26, 64, 64, 768),    # 641 rows for each of two rounds of tiles
])
def test_float32_tiles_follow_the_work(heights, c_in, c_out, rows):
    """float32 tiles hold one CU's share of the rows times column slices, 128 to 512 rows
    (whole rounds of 128), before the rule for large launches."""
    assert _wide_tiles(heights, c_in, c_out, 4)[1] == rows


@pytest.mark.parametrize("c_in,wide", [(4, False), (8, False), (12, False), (16, True), (20, False), (24, True),
                                       (36, True), (64, True), (68, False), (72, True), (132, False), (144, True),
                                       (256, True), (260, False)])
def test_float32_full_width_pads_a_third_at_most(c_in, wide):
    """k-steps of 16 channels (1, 2, 3, 4, 6, 8, 12 or 16 of them): layers that would pad more
    than a third, or fill less than one step, keep the general product."""
    gemm_wide = B.lib()._ZN3spc9gemm_wideEiiii
    gemm_wide.restype = ctypes.c_bool
    assert gemm_wide(c_in, 64, B.SPCONV_F32, B.SPCONV_F32) == wide
