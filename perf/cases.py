"""Performance cases of rngx: what its users have it do, over the range of sizes it is used at.

Kinds of case:
  plain   one rngx.generate / generate_u32 call of a seeded generator: the next `iters` values of
          each of its `n` streams into a device buffer;
  fresh   rngx.init and the first rngx.generate after it: a program that seeds a new generator for
          each job;
  batch   one rngx.generate_batch call: `m` independent streams of uneven lengths, packed;
  serve   `k` requests submitted together to the running server, waited for, read and released;
  stream  rngx.stream_to_host: `steps` steps of one value per stream into page-locked memory.

The paper's program runs n = 2^12 ... 2^24 streams for 10^2 ... 10^4 iterations, one iteration per
kernel call; the benchmark goes up to 2^26 streams, to tables of 4,096 streams of 2^10 ... 2^24
values, and to served requests of 2^12 ... 2^22 values on 2^20 resident streams.

The library has one generator and one server in a process. The state prepared last owns them, and
a pass takes the next values from them, as the one program that runs in a process does.
"""
import functools
import math

import numpy as np
import torch

from paper_1609_01257_amd import rngx

POOL_BYTES = 4 << 30
RESIDENT = 1 << 20
STAR = 2685821657736338717

# The output pool of the running server, kept until the server has stopped.
_server = {"pool": None}


def listed():
    return [
        # The smallest call of the paper's range, from a program that makes many of them (event
        # logging off): latency and launches.
        _plain("plain_4096x100", 4096, 100, logged=False),
        # The paper's smallest stream count at its largest iteration count.
        _plain("plain_4096x10000", 4096, 10000),
        # The plain method's small workload: seed 65,536 streams, take 64 values of each.
        {"name": "fresh_65536x64", "kind": "fresh", "n": 65536, "iters": 64, "u32": False,
         "star": False, "logged": True},
        # A stream count that is no power of two and odd: no row but the first is aligned.
        _plain("plain_1000003x256", 1000003, 256),
        # Scrambled 32-bit words for an odd count of streams.
        _plain("plain_262147x1000_u32_star", 262147, 1000, u32=True, star=True),
        # The benchmark's sweep, a middle size, 32-bit words.
        _plain("plain_4194304x256_u32", 1 << 22, 256, u32=True),
        # The benchmark's headline stream count, 32 GiB of values in one call.
        _plain("plain_67108864x64", 1 << 26, 64),
        # A handful of ragged streams, from anywhere in them: one small batched call.
        _batch("batch_3_small", 3, 12.0, 16.0, 1 << 20),
        # Some hundreds of ragged streams: an ordinary batched call.
        _batch("batch_256_medium", 256, 10.0, 17.0, 1 << 30),
        # The benchmark's batched table: 4,096 streams of 2^10 ... 2^24 values, from their start.
        _batch("batch_4096_large", 4096, 10.0, 24.0, 0),
        # Requests of the benchmark's served lengths arriving together at the server.
        {"name": "serve_32", "kind": "serve", "k": 32, "lo": 12.0, "hi": 22.0, "star": False},
        # The paper's streaming run: 32 MiB a step to the host, generation under the copies.
        {"name": "stream_4194304x8", "kind": "stream", "n": 1 << 22, "steps": 8, "u32": False,
         "star": False, "logged": True},
    ]


def _plain(name, n, iters, u32=False, star=False, logged=True):
    return {"name": name, "kind": "plain", "n": n, "iters": iters, "u32": u32, "star": star,
            "logged": logged}


def _batch(name, m, lo, hi, max_offset):
    return {"name": name, "kind": "batch", "m": m, "lo": lo, "hi": hi, "max_offset": max_offset,
            "star": False}


def draw(rng):
    kind = rng.choices(["plain", "fresh", "batch", "serve", "stream"], [8, 2, 6, 2, 2])[0]
    star = rng.random() < 0.25
    if kind in ("plain", "fresh"):
        n = _log_int(rng, 1 << 12, 1 << 26 if kind == "plain" else 1 << 22)
        n = rng.choice([n | 1, n, n & ~15])
        u32 = rng.random() < 0.4
        most = min(10000, (1 << 35) // (n * (4 if u32 else 8)))
        return {"kind": kind, "n": n, "iters": _log_int(rng, 1, most), "u32": u32, "star": star,
                "logged": rng.random() < 0.5 or kind == "fresh"}
    if kind == "batch":
        m = _log_int(rng, 1, 4096)
        lo = round(rng.uniform(4.0, 12.0), 2)
        hi = round(rng.uniform(lo + 1.0, 24.0), 2)
        while m * _mean_length(lo, hi) > 7.0e9:
            hi = round(hi - 0.25, 2)
        return {"kind": kind, "m": m, "lo": lo, "hi": hi,
                "max_offset": rng.choice([0, 1 << 20, 1 << 40]), "star": star}
    if kind == "serve":
        return {"kind": kind, "k": _log_int(rng, 1, 60), "lo": 12.0,
                "hi": round(rng.uniform(13.0, 22.0), 2), "star": star}
    n = _log_int(rng, 1 << 12, 1 << 22)
    n = rng.choice([n | 1, n, n & ~15])
    u32 = rng.random() < 0.4
    return {"kind": kind, "n": n, "steps": _log_int(rng, 2, min(100, (1 << 28) // (8 * n))),
            "u32": u32, "star": star, "logged": rng.random() < 0.5}


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _mean_length(lo, hi):
    return (2.0 ** hi - 2.0 ** lo) / (math.log(2.0) * (hi - lo))


def _lengths(case):
    """The lengths of a case's requests: floor(2^U[lo, hi)), the same for every seed."""
    count = case["m"] if case["kind"] == "batch" else case["k"]
    u = np.random.default_rng(1609).uniform(case["lo"], case["hi"], size=count)
    return np.floor(2.0 ** u).astype(np.uint64)


def _requests(case, seed):
    """(seeds, gids, offsets) of a batch, (stream ids) of served requests."""
    rng = np.random.default_rng(seed)
    if case["kind"] == "serve":
        return rng.integers(0, RESIDENT, size=case["k"], dtype=np.uint64).astype(np.uint32)
    m = case["m"]
    return (rng.integers(0, 2**64, size=m, dtype=np.uint64),
            rng.integers(0, 2**32, size=m, dtype=np.uint64).astype(np.uint32),
            rng.integers(0, case["max_offset"] + 1, size=m, dtype=np.uint64))


def _generator_seed(seed):
    return int(np.random.default_rng(seed).integers(0, 2**64, dtype=np.uint64))


def prepare(case, seed):
    kind = case["kind"]
    if _server["pool"] is not None:
        rngx.serve_stop()
        _server["pool"] = None
    rngx.set_scrambler(rngx.SCRAMBLE_STAR if case["star"] else rngx.SCRAMBLE_NONE)
    rngx.profile_enable(bool(case.get("logged", False)))
    s = {"kind": kind}
    if kind == "batch":
        lengths = _lengths(case)
        s["reqs"] = rngx.make_reqs(*_requests(case, seed), lengths)
        s["out"] = torch.empty(int(lengths.sum()), dtype=torch.int64, device="cuda")
        return s
    if kind == "serve":
        pool = torch.empty(POOL_BYTES // 8, dtype=torch.int64, device="cuda")
        rngx.serve_start(_generator_seed(seed), RESIDENT, pool, 4, 2048)
        _server["pool"] = pool
        s["ids"], s["lengths"] = _requests(case, seed), _lengths(case)
        return s
    n, dtype = case["n"], torch.int32 if case["u32"] else torch.int64
    s.update(n=n, seed=_generator_seed(seed), u32=case["u32"])
    if kind == "stream":
        s["steps"] = case["steps"]
        s["dev"] = [torch.empty(n, dtype=dtype, device="cuda") for _ in range(2)]
        s["host"] = torch.empty(n * case["steps"], dtype=dtype, pin_memory=True)
    else:
        s["iters"] = case["iters"]
        s["out"] = torch.empty(n * case["iters"], dtype=dtype, device="cuda")
    if kind != "fresh":
        rngx.init(s["seed"], n)
    return s


def run(state):
    kind = state["kind"]
    if kind == "batch":
        rngx.generate_batch(state["reqs"], state["out"])
        return state["out"]
    if kind == "serve":
        pool = _server["pool"]
        lengths = state["lengths"]
        tickets = rngx.serve_submit_many(state["ids"], lengths)
        values = []
        for ticket, length in zip(tickets.tolist(), lengths.tolist()):
            at = (rngx.serve_wait(ticket) - pool.data_ptr()) // 8
            values.append(pool[at:at + length])
        for ticket in tickets.tolist():
            rngx.serve_release(ticket)
        return values
    if kind == "stream":
        rngx.stream_to_host(state["steps"], 1, state["dev"][0], state["dev"][1], state["host"],
                            state["steps"], u32=state["u32"])
        return state["host"]
    if kind == "fresh":
        rngx.init(state["seed"], state["n"])
    (rngx.generate_u32 if state["u32"] else rngx.generate)(state["iters"], state["out"])
    return state["out"]


def work(case):
    """Each value written once; a plain call also reads and writes its 8-byte states once, a
    new generator only writes them."""
    if case["kind"] in ("batch", "serve"):
        return {"bytes": 8 * int(_lengths(case).sum()), "flops": 0}
    n, iters = case["n"], case.get("steps", case.get("iters"))
    states = 8 * n if case["kind"] == "fresh" else 16 * n
    return {"bytes": (4 if case["u32"] else 8) * n * iters + states, "flops": 0}


# The same values from the definitions of the generator and its seeding, in plain torch on 64-bit
# integers: what a first pass after prepare() returns.

def exact(case, seed):
    kind, star = case["kind"], case["star"]
    if kind == "batch":
        seeds, gids, offsets = _requests(case, seed)
        x = _jump(_initial(seeds, gids), offsets)
        return _word(_packed(x, _lengths(case)), star, False)
    if kind == "serve":
        ids, lengths = _requests(case, seed), _lengths(case)
        cursor, offsets = {}, []
        for g, length in zip(ids.tolist(), lengths.tolist()):
            offsets.append(cursor.get(g, 0))
            cursor[g] = offsets[-1] + length
        seeds = np.full(len(ids), _generator_seed(seed), dtype=np.uint64)
        x = _jump(_initial(seeds, ids), np.array(offsets, dtype=np.uint64))
        v = _word(_packed(x, lengths), star, False)
        return list(v.split(lengths.tolist()))
    n, rows = case["n"], case.get("steps", case.get("iters"))
    x = _initial(np.uint64(_generator_seed(seed)), torch.arange(n, device=_device()))
    out = torch.empty((rows, n), dtype=torch.int32 if case["u32"] else torch.int64,
                      device=_device())
    for k in range(rows):
        out[k] = _word(x, star, case["u32"])
        x = _step(x)
    return out.reshape(-1).cpu() if kind == "stream" else out.reshape(-1)


def _device():
    return "cuda" if torch.cuda.is_available() else "cpu"


def _right(x, k):
    """Logical shift of 64-bit words."""
    return (x >> k) & ((1 << (64 - k)) - 1)


def _step(x):
    x = x ^ (x << 21)
    x = x ^ _right(x, 35)
    return x ^ (x << 4)


def _word(x, star, u32):
    """In place for 64-bit words."""
    if star:
        x = x.clone() if u32 or x.numel() < (1 << 28) else x
        x *= STAR
    if u32:
        return (_right(x, 32) if star else x & 0xFFFFFFFF).to(torch.int32)
    return x


def _hash_low(a):
    m = 0xFFFFFFFF
    a = ((a + 0x7ed55d16) + (a << 12)) & m
    a = (a ^ 0xc761c23c) ^ (a >> 19)
    a = ((a + 0x165667b1) + (a << 5)) & m
    a = ((a + 0xd3a2646c) ^ (a << 9)) & m
    a = ((a + 0xfd7046c5) + (a << 3)) & m
    return (a ^ 0xb55a4f09) ^ (a >> 16)


def _hash_high(a):
    m = 0xFFFFFFFF
    a = (a ^ 61) ^ (a >> 16)
    a = (a + (a << 3)) & m
    a = a ^ (a >> 4)
    a = (a * 0x27d4eb2d) & m
    return a ^ (a >> 15)


def _initial(seeds, gids):
    """Initial states: the hashes of the paper's init kernel with the seed folded in."""
    seeds = np.atleast_1d(np.asarray(seeds, dtype=np.uint64))
    lo = torch.from_numpy((seeds & np.uint64(0xFFFFFFFF)).astype(np.int64)).to(_device())
    hi = torch.from_numpy((seeds >> np.uint64(32)).astype(np.int64)).to(_device())
    if not isinstance(gids, torch.Tensor):
        gids = torch.from_numpy(gids.astype(np.int64)).to(_device())
    low = _hash_low(gids ^ _hash_low(lo) ^ _hash_low(0))
    high = _hash_high(low ^ _hash_high(hi) ^ _hash_high(0))
    x = (high << 32) | low
    return torch.where(x == 0, torch.full_like(x, _signed(_hash_high(0) << 32)), x)


def _signed(v):
    return v - (1 << 64) if v >= 1 << 63 else v


@functools.lru_cache(maxsize=None)
def _power(b):
    """2^b steps as a linear map: 8 tables of 256 entries, one for each byte of a state."""
    unit = torch.tensor([_signed(1 << j) for j in range(64)], dtype=torch.int64, device=_device())
    col = _step(unit) if b == 0 else _apply(_power(b - 1), _apply(_power(b - 1), unit))
    tables = torch.zeros((8, 256), dtype=torch.int64, device=_device())
    value = torch.arange(256, device=_device())
    for q in range(8):
        for j in range(8):
            tables[q] ^= torch.where((value >> j) & 1 == 1, col[8 * q + j], 0)
    return tables


def _apply(tables, x):
    y = tables[0][x & 255]
    for q in range(1, 8):
        y ^= tables[q][(x >> (8 * q)) & 255]
    return y


def _jump(x, offsets):
    for b in range(int(offsets.max()).bit_length()):
        on = torch.from_numpy(((offsets >> np.uint64(b)) & np.uint64(1)).astype(bool))
        x = torch.where(on.to(x.device), _apply(_power(b), x), x)
    return x


def _packed(x, lengths):
    """lengths[j] values from state x[j] on, one stream after the other: each stream's known
    values, 2^b of them, give its next 2^b."""
    lengths = [int(v) for v in lengths]
    known, b = x[:, None], 0
    while known.shape[1] * 2 <= min(lengths):
        known = torch.cat([known, _apply(_power(b), known)], 1)
        b += 1
    out = torch.empty(sum(lengths), dtype=torch.int64, device=x.device)
    at = 0
    for j, length in enumerate(lengths):
        v, c = out[at:at + length], 1 << b
        v[:c] = known[j]
        while c < length:
            more = min(c, length - c)
            v[c:c + more] = _apply(_power(c.bit_length() - 1), v[:more])
            c += more
        at += length
    return out
