"""CPU check of the direct-to-LDS first load (load_global_m0_fresh) over the
block shapes of the compiled kernels, 2^b words with 2^e per lane: the 16-byte
form and the 4-byte form of data that is only 8-byte aligned."""
import numpy as np
import pytest

from test_host_indexing import dma_swz

SHAPES = [(8, 2), (9, 2), (10, 2), (9, 3), (10, 3), (11, 3), (12, 3), (13, 3), (10, 4), (12, 4), (14, 4)]


@pytest.mark.parametrize("unit", [4, 1])
@pytest.mark.parametrize("b,e", SHAPES)
def test_direct_lds_load_maps(b, e, unit):
    """Dwords (two a word, four a pair): every instruction fills 64 x unit
    consecutive dwords of its wave's window, each LDS dword is written once from
    inside the block, and the pair that a lane reads back is its own."""
    lanes, wave_words = 1 << (b - e), 64 << e
    assert lanes % 64 == 0
    held = np.full(2 << b, -1, dtype=np.int64)             # global dword held by each LDS dword
    lane = np.arange(64)
    step = 32 * unit                                       # words an instruction moves
    for wave in range(lanes // 64):
        for i in range(wave_words // step):
            win = wave * wave_words + step * i
            if unit == 4:
                pair = win // 2 + lane
                src = (4 * dma_swz(pair))[:, None] + np.arange(4)
            else:
                src = (4 * dma_swz(win // 2 + (lane >> 2)) + (lane & 3))[:, None]
            dst = (2 * win + unit * lane)[:, None] + np.arange(unit)   # the hardware's: base + lane x size
            assert src.min() >= 0 and src.max() < held.size and dst.max() < held.size
            assert (held[dst] == -1).all()
            held[dst] = src
    assert (held >= 0).all()
    tid = np.arange(lanes)
    for j in range(1 << (e - 1)):
        want = (tid << (e - 1)) + j
        for d in range(4):
            assert (held[4 * dma_swz(want) + d] == 4 * want + d).all()
