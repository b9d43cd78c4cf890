"""Answers written at any alignment by the split reduction, requests restaged
from any alignment, and synchronous reads on both sides of the sizes that go
through mapped host memory: bit-exact against the CPU oracle, with the bytes
around every answer row untouched."""
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


@pytest.mark.parametrize("n,row,B", [(2000, 1, 3), (1999, 15, 9), (640, 16, 5), (4097, 17, 40), (3001, 999, 24),
                                     (8192, 320, 7), (70, 33, 2)])
def test_unaligned_rows(n, row, B):
    import torch
    D = synth.uniform_db(n + row, n, row)
    req = synth.bernoulli_requests(n, B, n)
    want = oracle.pir_read(D, req, threads=4)
    nb = (n + 7) // 8
    with pir.PirDB(n, 1, row) as db:
        db.load(D)
        for splits in (0, 1, 3):
            for off, pad in ((0, 0), (1, 2), (3, 5), (4, 12), (16, 16)):
                db.set_plan(pir.KERNEL_MASK, 0, splits)
                say(f"n={n} row={row} B={B} splits={splits} off={off} pad={pad}")
                q = torch.full((B, nb + off + pad), 0xFF, dtype=torch.uint8, device="cuda")
                q[:, off:off + nb] = torch.from_numpy(req).cuda()
                big = torch.full((B + 1, row + off + pad), 0xA5, dtype=torch.uint8, device="cuda")
                db.read_async(q[:, off:off + nb], big[:B, off:off + row])
                torch.cuda.synchronize()
                got = big.cpu().numpy()
                assert_rows_equal(got[:B, off:off + row], want, f"splits={splits} off={off}")
                got[:B, off:off + row] = 0xA5
                assert (got == 0xA5).all()


# answer bytes and request bytes just below, at and above 512 KiB
@pytest.mark.parametrize("n,row,Bs", [(1000, 4096, (1, 127, 128, 129)), (3333, 1001, (523, 524)),
                                      (131072, 64, (31, 32, 33)), (131072 + 5, 48, (31, 32))])
def test_synchronous_reads_around_the_mapped_sizes(n, row, Bs):
    D = synth.uniform_db(n + row, n, row)
    with pir.PirDB(n, 1, row) as db:
        db.load(D)
        for B in Bs + Bs[:1]:
            req = synth.bernoulli_requests(B, B, n)
            seeds = synth.bernoulli_requests(B + 1, B, 256)
            want = oracle.pir_read(D, req, threads=8)
            say(f"n={n} row={row} B={B}")
            assert_rows_equal(db.read(req), want, f"B={B}")
            db.set_plan(pir.KERNEL_MASK, 0, 1)
            assert_rows_equal(db.read(req), want, f"B={B} one split")
            db.set_plan()
            assert_rows_equal(db.read_masked(req, seeds), oracle.apply_masks(want, seeds), f"B={B} masked")
