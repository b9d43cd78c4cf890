"""Preprocessed reads whose leaves share one launch, at sizes where it takes
one split, a few and many: bit-exact against the CPU oracle, for each table
form that a leaf's batch size chooses."""
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


@pytest.mark.parametrize("n,d,z,levels", [(512, 4, 1024, 2), (8192, 1, 64, 1), (1 << 15, 1, 256, 2), (1 << 15, 2, 1024, 1)])
def test_leaves_with_few_and_many_splits(n, d, z, levels):
    D = synth.uniform_db(n + d, n, d * z)
    with pir.PirDB(n, d, z) as db:
        db.load(D)
        db.preprocess(levels, min_batch=1)
        for B in (40, 260, 700, 1100, 2048):
            req = synth.bernoulli_requests(B + n, B, n)
            say(f"n={n} row={d * z} levels={levels} B={B}")
            rows = np.unique(np.linspace(0, B - 1, 40).round().astype(np.int64))
            assert_rows_equal(db.read(req)[rows], oracle.pir_read(D, req[rows], threads=8), f"B={B}")
