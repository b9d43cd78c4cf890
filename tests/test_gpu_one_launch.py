"""The one-launch kernel of small databases at the edges of its steps (256 and
1024 buckets), its 64-byte columns, its request tiles and its range, with
aligned, unaligned and masked answers: bit-exact against the CPU oracle."""
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


@pytest.mark.parametrize("n,row", [(1, 16), (15, 3), (16, 64), (33, 80), (255, 999), (257, 4096), (1024, 4096), (1025, 65),
                                   (4096, 48), (5000, 1040)])
def test_every_tile_and_row(n, row):
    import torch
    D = synth.uniform_db(n + row, n, row)
    nb = (n + 7) // 8
    with pir.PirDB(n, 1, row) as db:
        db.load(D)
        for B in (1, 2, 3, 5, 8, 21):
            req = synth.bernoulli_requests(n + B, B, n)
            req[:, -1] |= np.uint8(0xFF << (n - 1) % 8 + 1 & 0xFF)   # bits past n are not looked at
            want = oracle.pir_read(D, req, threads=4)
            seeds = synth.uniform_bytes(B, B * 32).reshape(B, 32)
            for plan in ((), (pir.KERNEL_MASK, 1, 0, 4, pir.PLAN_ONE_LAUNCH), (pir.KERNEL_MASK, 2, 3, 0, pir.PLAN_ONE_LAUNCH),
                         (pir.KERNEL_MASK, 4, 1, 4, pir.PLAN_ONE_LAUNCH), (pir.KERNEL_MASK, 0, 0, 0, pir.PLAN_ONE_LAUNCH)):
                db.set_plan(*plan)
                say(f"n={n} row={row} B={B} plan={plan} tile={db.get_plan(B).tile} flags={db.get_plan(B).flags}")
                assert_rows_equal(db.read(req), want, f"{plan} sync")
                assert_rows_equal(db.read_masked(req, seeds), oracle.apply_masks(want, seeds), f"{plan} masked")
                q = torch.zeros((B, nb + 3), dtype=torch.uint8, device="cuda")[:, 1:1 + nb]
                q.copy_(torch.from_numpy(req))
                big = torch.full((B, row + 7), 0xA5, dtype=torch.uint8, device="cuda")
                db.profile_enable(B == 2)                        # the kernel's end event then is the profile's
                db.read_async(q, big[:, 3:3 + row])
                torch.cuda.synchronize()
                db.profile_enable(False)
                got = big.cpu().numpy()
                assert_rows_equal(got[:, 3:3 + row], want, f"{plan} async")
                assert (got[:, :3] == 0xA5).all() and (got[:, 3 + row:] == 0xA5).all()


def test_range_of_the_automatic_choice():
    for n, row, one in ((1024, 4096, (1, 2, 4, 8)), (1025, 4096, (1, 2, 4)), (4096, 4096, (1, 2)), (4096, 4112, ()),
                        (4097, 64, ()), (2048, 8192, (1, 2, 4)), (16, 16, (1, 8))):
        with pir.PirDB(n, 1, row) as db:
            for B in (1, 2, 4, 8, 9):
                p = db.get_plan(B)
                assert (p.flags == pir.PLAN_ONE_LAUNCH and p.splits == 1) == (B in one or (n == 16 and B < 9)), (n, row, B)
            for kind, tile, unroll, flags in ((pir.KERNEL_MASK, 16, 4, 0), (pir.KERNEL_MASK, 8, 8, 0), (pir.KERNEL_SKIP, 8, 4, 0),
                                              (pir.KERNEL_MASK, 8, 4, pir.PLAN_SHARED_COLUMN)):
                db.set_plan(kind, tile, 3, unroll, flags | pir.PLAN_ONE_LAUNCH)   # the plan without the flag
                p = db.get_plan(4)
                assert (p.kind, p.tile, p.unroll, p.flags) == (kind, tile, unroll, flags)
            db.set_plan()
