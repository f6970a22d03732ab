"""Device memory of the on-chip Krylov runs, on the CPU: the blocks of tagged
words and of plain values, for every kind of run that can follow another on one
grid's buffers.  A tag's place never holds anything but tags, so a word left
behind by an earlier run is never taken for one that has arrived."""
import ctypes
import os

import numpy as np
import pytest

from paper_1711_04060_amd import pf
from test_chip_tiles import GMAX, NT, Geom, partition

SUMS = 2 * 5 * (GMAX + 8) * 16 + GMAX * 8


class Space(ctypes.Structure):
    _fields_ = [(n, ctypes.c_size_t) for n in ("tagged", "plain", "face", "xtile")]


def space(ge, kz, elem):
    if not os.path.exists(pf.LIB_PATH):
        pytest.skip("library not built")
    f = getattr(ctypes.CDLL(pf.LIB_PATH), "_ZN3pfk10chip_spaceERKNS_8ChipGeomEim")
    f.restype, f.argtypes = Space, [ctypes.POINTER(Geom), ctypes.c_int, ctypes.c_size_t]
    return f(ctypes.byref(ge), kz, elem)


@pytest.mark.parametrize("elem", [4, 8])
@pytest.mark.parametrize("n", [(33, 33, 33), (65, 65, 65), (65, 40, 51), (97, 97, 97), (113, 113, 113), (129, 129, 129)])
def test_tags_and_plain_values_have_blocks_of_their_own(n, elem):
    seen = 0
    for cap in (GMAX, 128, 40):
        for lim in (8, 16):
            ge = partition(*n, 0, cap, lim)
            for kz in (4, 8, 16):
                if ge.KZ == 0 or kz < ge.KZ or kz > lim:   # a batch may use a larger instance than a member needs
                    continue
                seen += 1
                m = space(ge, kz, elem)
                assert m.tagged >= SUMS and m.face % 256 == 0 and m.xtile % 256 == 0
                words = 2 * ge.G * ge.fstride
                if kz <= 8:     # {value, tag} words only: 16 bytes of FP64 {lo, tag, hi, tag}, 8 of FP32 {v, tag}
                    assert m.plain == 0 and m.face >= SUMS and m.face + words * 2 * elem <= m.tagged
                    at = m.face + 2 * elem * np.arange(words)
                    tags = np.concatenate([at + 4, at + 12]) if elem == 8 else at + 4
                    assert ((tags // 4) % 2 == 1).all()    # the odd words, as of every other run
                else:           # no value without a tag in the tagged block
                    assert m.plain > 0 and m.face + words * elem <= m.xtile
                    assert m.xtile + ge.G * kz * NT * elem <= m.plain
    assert seen
