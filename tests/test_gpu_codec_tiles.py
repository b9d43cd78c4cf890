"""The device encoder of interest vectors at the edges of its tiles and of the
part of a body that comes by mapped memory: byte for byte the oracle's."""
import ctypes

import numpy as np
import pytest

import oracle
import paper_2001_08250_amd as pir
import synth
from helpers import gpu_available, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not gpu_available():
        pytest.skip("no GPU")


# one and two tiles of 1024 words and a bit more; bodies around the 64 KiB that
# come by mapped memory (a full vector of m bits takes m bits, the worst
# density m = 3 c about 1.4 m)
@pytest.mark.parametrize("m,every", [(32767, 5), (32768, 1), (32769, 40000), (65536 + 33, 64), (8 * 65536 - 1, 1),
                                     (8 * 65536 + 1, 1), (3 << 20, 3)])
def test_tiles_and_long_bodies(m, every):
    n, d, z = 16, 1, 16
    with pir.PirDB(n, d, z) as db:
        db.load(synth.uniform_db(11, n, d * z))
        db.interest_config(m, 3)
        for start in (0, every - 1, m - 1):          # each epoch's bits end or begin at a tile's edge
            pos = np.arange(start, m, every, dtype=np.uint32)
            db.interest_add(pos)
            db.commit()
            say(f"m={m} every={every} start={start}")
            v = np.zeros(m, dtype=np.uint8)
            v[pos] = 1
            want = oracle.iv_encode(np.packbits(v, bitorder="little"), m)
            for _ in range(2):                        # the passes leave their state as they found it
                assert db.interest_encoded(db.epoch) == want
            small = np.zeros(len(want) - 1, dtype=np.uint8)
            size = ctypes.c_uint64(0)
            for out, cap, rc in ((None, 0, pir.PIR_OK), (small.ctypes.data_as(ctypes.POINTER(ctypes.c_uint8)),
                                                         small.size, pir.PIR_EINVAL)):
                assert pir.lib().pir_interest_delta_encoded(db.h, db.epoch, out, cap, ctypes.byref(size)) == rc
                assert size.value == len(want)
            assert not small.any()
