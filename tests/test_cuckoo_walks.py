"""Long cuckoo walks (more evictions than one settling of the bytes takes,
walks that return to their slots, dropped messages) against the oracle."""
import numpy as np
import pytest

import oracle
import paper_2001_08250_amd as pir
import synth


@pytest.mark.parametrize("n,d,z,buckets,count,capacity,kicks", [
    (64, 4, 5, 64, 300, 0, 3000),       # every slot full: walks of 3000 over 256 slots
    (400, 2, 16, 400, 840, 0, 2000),    # more slots than a settling holds
    (300, 4, 8, 3, 60, 0, 500),         # a few buckets that the same writes fill
    (300, 4, 8, 6, 400, 20, 37),        # with collection of the oldest
    (9, 1, 3, 9, 40, 0, 1), (5, 1, 1, 1, 12, 0, 0),
])
def test_long_walks_match_the_oracle(n, d, z, buckets, count, capacity, kicks):
    ids, b1, b2, pay = synth.write_ops(n + count, count, buckets, z)
    ref = oracle.Cuckoo(n, d, z, capacity=capacity, seed=3, max_kicks=kicks)
    mine = pir.Cuckoo(None, capacity=capacity, seed=3, max_kicks=kicks, shape=(n, d, z))
    for part in np.array_split(np.arange(count), 5):
        st, dr = mine.insert_many(ids[part], b1[part], b2[part], pay[part])
        st_ref, dr_ref = ref.insert_many(ids[part], b1[part], b2[part], pay[part])
        assert np.array_equal(st, st_ref) and np.array_equal(dr, dr_ref)
        assert np.array_equal(mine.table(), ref.table())
        for x, y in zip(mine.slots(), ref.slots()):
            assert np.array_equal(x, y)
        assert mine.live() == ref.live()
