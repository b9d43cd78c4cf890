"""The matrix-core read kernel against the CPU oracle (bit-exact: counts are
whole numbers below 2^24 in fp32, so the tolerance is 0), and the automatic
choice of it against the masked kernel."""
import numpy as np
import pytest

import oracle
import paper_2001_08250_amd as pir
import synth
from helpers import assert_rows_equal, gpu_available, say

pytestmark = pytest.mark.gpu

TILES = (32, 64, 96, 128)


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not gpu_available():
        pytest.skip("no GPU")


# edges of the 256 / 512 bucket chunks, of the 64 / 128 / 256 byte column
# tiles, of 32-bucket words and of 32-request tiles
@pytest.mark.parametrize("n,d,z", [(1, 1, 16), (31, 3, 20), (257, 2, 520), (1000, 1, 8), (2049, 8, 40), (3000, 1, 4000)])
def test_every_tile_at_its_edges(n, d, z):
    D = synth.uniform_db(n * 7 + d, n, d * z)
    with pir.PirDB(n, d, z) as db:
        db.load(D)
        for B in (1, 32, 33, 65, 97, 129, 300):
            req = synth.bernoulli_requests(n + B, B, n)
            want = oracle.pir_read(D, req, threads=8)
            for tile in TILES:
                for splits in (0, 1, 3):
                    say(f"n={n} d={d} z={z} B={B} tile={tile} splits={splits}")
                    db.set_plan(pir.KERNEL_MFMA, tile, splits, 4, 0)
                    assert_rows_equal(db.read(req), want, f"B={B} tile={tile} splits={splits}")


@pytest.mark.parametrize("n", [(1 << 20) - 33, (1 << 20), (1 << 20) + 4097, (1 << 21) + 5])
def test_counts_up_to_the_split_limit(n):
    """All-ones requests and rows: every count is as large as it can be. One
    split holds at most 2^20 buckets, a forced smaller count is raised."""
    row = 16
    D = np.full((n, row), 255, np.uint8)
    D[:, 1] = 0x55
    D[::2, 2] = 0
    want = np.full(row, 255 if n & 1 else 0, np.uint8)
    want[1] = 0x55 if n & 1 else 0
    want[2] = 255 if (n // 2) & 1 else 0
    q = np.full((40, (n + 7) // 8), 255, np.uint8)
    with pir.PirDB(n, 1, row) as db:
        db.load(D)
        for tile in TILES:
            for splits in (1, 0):
                db.set_plan(pir.KERNEL_MFMA, tile, splits, 4, 0)
                p = db.get_plan(40)
                say(f"n={n} tile={tile} splits={p.splits}")
                assert p.splits * (1 << 20) >= n
                assert (db.read(q) == want).all(), (tile, splits)


@pytest.mark.parametrize("n,d,z", [(1000, 3, 100), (2000, 4, 260), (4128, 1, 512), (8160, 2, 64), (5000, 1, 48), (8200, 1, 2000), (70000, 1, 64)])
def test_automatic_choice_equals_the_masked_kernel(n, d, z):
    """Pitched and unaligned requests and answers, masked answers, from the
    smallest batch that takes the matrix cores to beyond the tables'."""
    import torch
    dev = torch.device("cuda:0")
    D = synth.uniform_db(n + 3, n, d * z)
    nb = (n + 7) // 8
    with pir.PirDB(n, d, z) as db:
        db.load(D)
        kinds = set()
        for B in (8, 9, 17, 40, 100, 128, 129, 256, 257, 520):
            req = torch.from_numpy(synth.bernoulli_requests(B, B, n)).to(dev)
            q = torch.zeros((B, nb + 16 + 3), dtype=torch.uint8, device=dev)[:, 1:1 + nb]
            q.copy_(req)
            big = torch.zeros((B, d * z + 37), dtype=torch.uint8, device=dev)
            out, ref = big[:, 5:5 + d * z], torch.zeros((B, d * z), dtype=torch.uint8, device=dev)
            db.set_plan()
            kinds.add(db.get_plan(B).kind)
            say(f"n={n} d={d} z={z} B={B} kind={db.get_plan(B).kind}")
            db.read_async(q, out)
            plain, near = torch.zeros_like(ref), torch.zeros_like(ref)
            db.read_async(req, plain)        # in place where rows are whole words (4128 and 8160 buckets)
            at4 = torch.zeros((B, nb + 8), dtype=torch.uint8, device=dev)[:, 4:4 + nb]
            at4.copy_(req)
            db.read_async(at4, near)
            db.set_plan(pir.KERNEL_MASK)
            db.read_async(req, ref)
            torch.cuda.synchronize()
            assert torch.equal(out, ref) and torch.equal(plain, ref) and torch.equal(near, ref), B
            assert not big[:, :5].any() and not big[:, 5 + d * z:].any()
        assert pir.KERNEL_MFMA in kinds


def test_other_plans_are_refused_and_saved_ones_load(tmp_path):
    n, d, z = 4096, 1, 512
    with pir.PirDB(n, d, z) as db:
        for tile, unroll, flags in ((16, 4, 0), (160, 4, 0), (64, 8, 0), (64, 4, pir.PLAN_PAIRS)):
            with pytest.raises(pir.PirError):
                db.set_plan(pir.KERNEL_MFMA, tile, 0, unroll, flags)
        path = tmp_path / "plans.json"
        path.write_text('[\n {"n": 4096, "bclass": 64, "stride": 512, "kind": 5, "tile": 64, "splits": 3, '
                        '"unroll": 4, "flags": 0, "us": 20.0}\n]\n')
        assert pir.lib().pir_tune_load(str(path).encode()) == 0
        bad = tmp_path / "bad.json"
        bad.write_text(path.read_text().replace('"tile": 64', '"tile": 48'))
        assert pir.lib().pir_tune_load(str(bad).encode()) != 0
        D = synth.uniform_db(9, n, d * z)
        req = synth.bernoulli_requests(10, 60, n)
        db.load(D)
        say("saved plan", db.get_plan(60).kind, db.get_plan(60).splits)
        assert_rows_equal(db.read(req), oracle.pir_read(D, req, threads=8), "saved plan")
