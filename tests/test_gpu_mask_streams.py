"""Batches of up to 8 requests around the sizes where the masked kernel's
automatic schedule changes: databases that the caches hold, streamed ones and
ones read past the caches (nontemporal loads), narrow rows on the matrix cores.
Bit-exact against the CPU oracle."""
import numpy as np
import pytest

import oracle
import paper_2001_08250_amd as pir
import synth
from helpers import assert_rows_equal, gpu_available, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not gpu_available():
        pytest.skip("no GPU")


# bytes of n rows: 64 MiB, just above it, just above 256 MiB with a ragged last
# chunk and a last word of one bucket; narrow rows from 16 MiB on
@pytest.mark.parametrize("n,row", [(1 << 16, 1024), ((1 << 16) + 31, 1040), ((1 << 18) + 33, 1030), ((1 << 19) + 1, 520),
                                   ((1 << 18) + 5, 64), ((1 << 16) + 7, 256)])
def test_small_batches_around_the_streaming_sizes(n, row):
    D = synth.uniform_db(n + row, n, row)
    req = synth.bernoulli_requests(n, 8, n)
    want = oracle.pir_read(D, req, threads=8)
    with pir.PirDB(n, 1, row) as db:
        db.load(D)
        for B in (1, 2, 3, 5, 8):
            p = db.get_plan(B)
            say(f"n={n} row={row} B={B} kind={p.kind} tile={p.tile} unroll={p.unroll} splits={p.splits}")
            assert_rows_equal(db.read(req[:B]), want[:B], f"B={B}")
        # one request tile read once, by every column layout of both families
        for kind in (pir.KERNEL_MASK, pir.KERNEL_SKIP):
            for tile, unroll, flags in ((8, 4, 0), (8, 8, pir.PLAN_SHARED_COLUMN), (4, 4, pir.PLAN_SHARED_COLUMN), (16, 16, 0)):
                db.set_plan(kind, tile, 0, unroll, flags)
                assert_rows_equal(db.read(req), want, f"kind={kind} tile={tile} unroll={unroll} flags={flags}")
