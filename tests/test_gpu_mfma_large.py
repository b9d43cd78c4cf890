"""The matrix-core kernel over a database past the last-level cache (each tile's
nontemporal form), at rows and request pitches too long for its 32-bit offsets,
and as the leaves' kernel: bit-exact against the CPU oracle."""
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


def test_one_request_tile_past_the_cache():
    n, row = (1 << 18) + 33, 1030                       # 260 MiB, ragged in both directions
    D = synth.uniform_db(n, n, row)
    req = synth.bernoulli_requests(n + 1, 128, n)
    want = oracle.pir_read(D, req, threads=8)
    with pir.PirDB(n, 1, row) as db:
        db.load(D)
        for tile in (32, 64, 96, 128):
            for B in (tile - 31, tile):
                for splits in (0, 1):
                    say(f"tile={tile} B={B} splits={splits}")
                    db.set_plan(pir.KERNEL_MFMA, tile, splits, 4, 0)
                    assert_rows_equal(db.read(req[:B]), want[:B], f"tile={tile} B={B} splits={splits}")
        db.set_plan()
        for B in (9, 33, 64, 128):
            p = db.get_plan(B)
            say(f"auto B={B} kind={p.kind} tile={p.tile} splits={p.splits}")
            assert p.kind == pir.KERNEL_MFMA
            assert_rows_equal(db.read(req[:B]), want[:B], f"auto B={B}")


def test_rows_too_long_for_the_kernel():
    n, row = 3, (4 << 20) + 16
    D = synth.uniform_db(5, n, row)
    with pir.PirDB(n, 1, row) as db:
        db.load(D)
        for tile in (64, 96, 128):
            with pytest.raises(pir.PirError):
                db.set_plan(pir.KERNEL_MFMA, tile, 0, 4, 0)
        for B in (9, 40):
            req = synth.bernoulli_requests(B, B, n)
            say(f"row={row} B={B} kind={db.get_plan(B).kind}")
            assert db.get_plan(B).kind != pir.KERNEL_MFMA
            assert_rows_equal(db.read(req), oracle.pir_read(D, req, threads=8), f"B={B}")


def test_request_pitch_too_long_for_the_kernel():
    import torch
    n, row, B = 1024, 512, 9
    D = synth.uniform_db(6, n, row)
    req = synth.bernoulli_requests(7, B, n)
    want = oracle.pir_read(D, req)
    q = torch.zeros((B, 16 << 20), dtype=torch.uint8, device="cuda")[:, :n // 8]
    q.copy_(torch.from_numpy(req))
    out = torch.zeros((B, row), dtype=torch.uint8, device="cuda")
    with pir.PirDB(n, 1, row) as db:
        db.load(D)
        for plan in ((), (pir.KERNEL_MFMA, 128, 0, 4, 0), (pir.KERNEL_MFMA, 64, 0, 4, 0)):
            db.set_plan(*plan)
            say(f"pitch={q.stride(0)} plan={plan}")
            out.zero_()
            db.read_async(q, out)
            torch.cuda.synchronize()
            assert_rows_equal(out.cpu().numpy(), want, f"plan={plan}")


@pytest.mark.parametrize("tile", [32, 128])
def test_as_the_kernel_of_strassen_leaves(tile):
    n, row, B = 3000, 1024, 150
    D = synth.uniform_db(8, n, row)
    req = synth.bernoulli_requests(9, B, n)
    want = oracle.pir_read(D, req, threads=8)
    with pir.PirDB(n, 1, row) as db:
        db.load(D)
        db.set_plan(pir.KERNEL_MFMA, tile, 0, 4, 0)
        for levels in (1, 2):
            db.preprocess(levels, min_batch=1)
            say(f"levels={levels} tile={tile}")
            assert_rows_equal(db.read(req), want, f"levels={levels} tile={tile}")
