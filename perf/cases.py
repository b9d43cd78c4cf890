"""Workloads of the XOR-PIR server path, as a Talek server's program runs them.

Sizes come from the store sizes of the paper's cost table (10K, 100K and 1M
messages of 1 KiB in buckets of d = 4), from synth/configs.py and from the
ragged shapes that the tests use. Requests are uniform bit vectors and buckets
uniform bytes, which is all a server ever sees.

A case's ``op`` names what one pass does:

    read      one batch of device-resident request rows (pir_read_batch_async);
              ``levels`` > 0 answers it through Strassen leaves, ``odd`` starts
              rows one byte off their alignment at odd pitches
    host      one batch through the synchronous call, host rows in and out
    leader    a leader of serialized PIR: its own masked answers, then their
              combination with two followers' masked answers
    step      one served batch: B/10 cuckoo writes with their interest bits, the
              commit that publishes them, the read, the interest vector
    stream    uneven batches with sizes drawn from 1 .. top, as one stream
    updates   one write interval's GetUpdates: its interest bits, the commit, the
              compressed delta
"""
import math

import numpy as np
import torch

import paper_2001_08250_amd as pir
import synth
from synth import configs

GiB = 1 << 30
OPS = ("read", "host", "leader", "step", "stream", "updates")


def _case(name, op, n=0, d=4, z=1024, B=0, levels=0, odd=False, batches=0, top=0, items=0, messages=0):
    c = {"op": op, "n": n, "d": d, "z": z, "B": B, "levels": levels, "odd": odd, "batches": batches, "top": top,
         "items": items, "messages": messages}
    return {"name": name, **c} if name else c


def listed():
    return [
        # The smallest configuration: launch latency and host calls.
        _case("c1 read 8 of 4 MiB", "read", n=1024, B=8),
        # One read over the paper's 10K-message store, host rows in and out (rows of 329 bytes).
        _case("host read 1 of 10 MiB", "host", n=2632, B=1),
        # One read over the paper's 1M-message store: a lone client's latency, bound by memory.
        _case("read 1 of 1 GiB", "read", n=1 << 18, B=1),
        # A serving batch at a modest load over the same store.
        _case("read 64 of 1 GiB", "read", n=1 << 18, B=64),
        # Buckets of 999 bytes, rows off their alignment, a 100K-message store.
        _case("ragged read 24 of 25 MiB", "read", n=26_317, d=3, z=333, B=24, odd=True),
        # The 256 MiB configuration's batch.
        _case("c2 read 256 of 256 MiB", "read", n=65_536, B=256),
        # Serialized PIR at a leader.
        _case("leader 128 of 256 MiB", "leader", n=65_536, B=128),
        # The whole server step on the 256 MiB cuckoo-filled configuration.
        _case("c2 step 256 of 256 MiB", "step", n=65_536, B=256, items=200_000),
        # Uneven batches over the same store.
        _case("stream 12 x 1..1024 of 256 MiB", "stream", n=65_536, batches=12, top=1024),
        # A large plain batch over 8 KiB buckets.
        _case("read 1000 of 1 GiB", "read", n=1 << 17, d=2, z=4096, B=1000),
        # The largest: 2048 reads of 2 GiB through two levels of Strassen leaves.
        _case("leaves 2048 of 2 GiB", "read", n=1 << 18, d=2, z=4096, B=2048, levels=2),
        # GetUpdates of the paper's 100K-message store.
        _case("updates of 100K messages", "updates", n=1024, d=1, z=64, messages=100_000),
    ]


def _log(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    op = rng.choice(("read", "read", "read", "read", "leaves") + OPS[1:])
    if op == "updates":
        return _case(None, "updates", n=1024, d=1, z=64, messages=_log(rng, 10_000, 400_000))
    if op == "leaves":
        d, z = rng.choice(((4, 1024), (2, 4096), (1, 2048), (4, 512)))
        n = _log(rng, 32_768, GiB // (d * z))
        return _case(None, "read", n=n, d=d, z=z, B=rng.randint(1024, 2048), levels=2)
    if op == "step":
        return _case(None, "step", n=_log(rng, 4096, 65_536) // 32 * 32, B=_log(rng, 8, 512), items=-1)
    d, z = rng.choice(((4, 1024), (4, 1024), (4, 1024), (2, 4096), (3, 333), (1, 256), (8, 40), (1, 2048)))
    n = _log(rng, 1000, min(1 << 18, GiB // (d * z)))
    B = _log(rng, 1, 2048)
    if op == "stream":  # whole words and whole 16-byte rows, as the call asks for
        d, z = rng.choice(((4, 1024), (2, 4096), (1, 256)))
        n = _log(rng, 1024, 1 << 16) // 32 * 32
        return _case(None, "stream", n=n, d=d, z=z, batches=rng.randint(4, 24), top=_log(rng, 32, 1024))
    if op == "leader":
        return _case(None, "leader", n=n, d=4, z=_log(rng, 4, 256) * 4, B=min(B, 512))
    if op == "host":
        return _case(None, "host", n=n, d=d, z=z, B=min(B, 256))
    return _case(None, "read", n=n, d=d, z=z, B=B, odd=rng.random() < 0.25)


def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _bytes(gen, *shape):
    return torch.randint(0, 256, shape, dtype=torch.uint8, device="cuda", generator=gen)


def _items(case):
    """Messages in a cuckoo-filled store: the configuration's, or its load of 3/4."""
    return case["items"] if case["items"] > 0 else 3 * case["n"] * case["d"] // 4


def _sizes(case):
    """Batch sizes of a stream, the same for every seed."""
    return synth.batch_sizes(configs.C3.batch_seed, case["batches"], 1, case["top"])


def _rows(case):
    """Request rows of a case."""
    return int(_sizes(case).sum()) if case["op"] == "stream" else case["B"]


def _requests(case, seed):
    rb = (case["n"] + 7) // 8
    return _bytes(_gen(3 * seed + 1), _rows(case), rb)


def _database(case, seed):
    return _bytes(_gen(3 * seed), case["n"], case["d"] * case["z"])


def _updates_shape(case):
    return configs.getupdates_shape(case["messages"])


def _positions(case, seed):
    """Interest bits of one pass's writes."""
    if case["op"] == "updates":
        s = _updates_shape(case)
        return synth.interest_positions(seed, s["per_interval"], s["k"], s["m_bits"])
    return synth.interest_positions(seed, -(-case["B"] // 10), 6, pir.IV_DEFAULT_BITS)


def prepare(case, seed):
    op, n, d, z = case["op"], case["n"], case["d"], case["z"]
    db = pir.PirDB(n, d, z)
    s = {"op": op, "db": db}
    if op == "updates":
        shape = _updates_shape(case)
        db.interest_config(shape["m_bits"], shape["window"])
        s["pos"] = _positions(case, seed)
        # the client's buffer: the header and the longest possible code of an interval's bits
        c = shape["per_interval"]
        k = int(math.log2(max(1, shape["m_bits"] // (c + 1))))
        s["delta"] = np.zeros(24 + (c * (k + 1) + (shape["m_bits"] >> k) + 7) // 8, dtype=np.uint8)
        return s
    if op == "step":
        items, w = _items(case), -(-case["B"] // 10)
        table = pir.Cuckoo(db, capacity=items, seed=seed, max_kicks=configs.CUCKOO_MAX_KICKS)
        ids, b1, b2, payload = synth.write_ops(seed, items + w, n, z)
        table.insert_many(ids[:items], b1[:items], b2[:items], payload[:items])
        table.stage()
        db.commit()
        s.update(table=table, writes=(ids[items:], b1[items:], b2[items:], payload[items:]),
                 pos=_positions(case, seed), iv=torch.empty(pir.IV_DEFAULT_BITS // 8, dtype=torch.uint8, device="cuda"))
    else:
        db.load(_database(case, seed).cpu().numpy())
    if case["levels"]:
        db.preprocess(case["levels"])
    q = _requests(case, seed)
    B = q.shape[0]
    if op == "host":
        s["q"] = q.cpu().numpy()
        return s
    out = torch.empty((B, d * z), dtype=torch.uint8, device="cuda")
    if case["odd"]:
        buf = torch.zeros((B, q.shape[1] + 3), dtype=torch.uint8, device="cuda")
        buf[:, 1:1 + q.shape[1]] = q
        q = buf[:, 1:1 + q.shape[1]]
        out = torch.empty((B, d * z + 5), dtype=torch.uint8, device="cuda")[:, 1:1 + d * z]
    s.update(q=q, out=out)
    if op == "stream":
        s["sizes"] = _sizes(case)
    if op == "leader":
        gen = _gen(3 * seed + 2)
        s["seeds"] = _bytes(gen, B, 32)
        s["others"] = [_bytes(gen, B, d * z) for _ in range(2)]
        s["combined"] = torch.empty_like(out)
    return s


def run(s):
    op, db = s["op"], s["db"]
    if op == "host":
        return {"resp": db.read(s["q"])}
    if op == "updates":
        db.interest_add(s["pos"])
        epoch = db.commit()
        code = db.interest_encoded(epoch)
        s["delta"][:len(code)] = np.frombuffer(code, dtype=np.uint8)
        return {"delta": s["delta"], "bytes": len(code)}
    if op == "stream":
        db.read_stream_async(s["q"], s["sizes"], s["out"])
        return {"resp": s["out"]}
    if op == "leader":
        db.read_masked_async(s["q"], s["seeds"], s["out"])
        pir.xor_combine_async(s["combined"], [s["out"], *s["others"]])
        return {"masked": s["out"], "combined": s["combined"]}
    if op == "step":
        s["table"].insert_many(*s["writes"])
        s["table"].stage()
        db.interest_add(s["pos"])
        db.commit()
    db.read_async(s["q"], s["out"])
    if op == "step":
        stream = int(torch.cuda.current_stream().cuda_stream)
        rc = pir.pir_interest_vector_async(db.h, s["iv"].data_ptr(), s["iv"].numel(), stream)
        if rc != pir.PIR_OK:
            raise RuntimeError(pir.strerror(rc))
        return {"resp": s["out"], "interest": s["iv"]}
    return {"resp": s["out"]}


def work(case):
    """Bytes: the database, requests and answers once. Flops: the 32-bit XORs of
    the plain method, half of all (request, bucket, word) terms."""
    if case["op"] == "updates":
        s = _updates_shape(case)
        # the window's deltas, the new delta and the new vector, the positions
        return {"bytes": (s["window"] + 2) * s["m_bits"] / 8 + 4 * s["per_interval"], "flops": 0}
    n, row = case["n"], case["d"] * case["z"]
    B = _rows(case)
    b = n * row + B * ((n + 7) // 8) + B * row
    if case["op"] == "leader":  # seeds, the followers' rows and the combined ones
        b += B * 32 + 3 * B * row
    if case["op"] == "step":
        b += -(-B // 10) * case["z"] + pir.IV_DEFAULT_BITS // 8
    return {"bytes": b, "flops": B * n * row / 8}


def _product(q, D, n):
    """The rows of q (request bytes) times D over GF(2), as a float product of
    bits whose sums stay far below 2^24, in blocks of buckets."""
    B, row = q.shape[0], D.shape[1]
    bit = torch.arange(8, device="cuda", dtype=torch.uint8)
    bits = lambda x: ((x.unsqueeze(-1) >> bit) & 1).reshape(x.shape[0], -1)  # noqa: E731
    out = torch.zeros((B, row * 8), dtype=torch.uint8, device="cuda")
    step = max(8, min(8192, (1 << 28) // (row * 8)) // 8 * 8)
    for k in range(0, n, step):
        d = bits(D[k:k + step]).float()
        a = bits(q[:, k // 8:k // 8 + step // 8])[:, :d.shape[0]].float()
        out ^= (a @ d).to(torch.int32).to(torch.uint8) & 1
    return (out.reshape(B, row, 8) << bit).sum(-1, dtype=torch.uint8)


def exact(case, seed):
    op = case["op"]
    if op not in ("read", "host", "stream"):  # keystreams, cuckoo placement and codes: bytes, compared as they are
        return None
    resp = _product(_requests(case, seed), _database(case, seed), case["n"])
    return {"resp": resp.cpu().numpy() if op == "host" else resp}
