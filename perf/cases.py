"""The work this framework's users have it do, as timed cases through its public entry points.

A case is a dict of plain values: the entry point (``op``), the algorithm (``algo``; ``mixed``
for per-message algorithm ids), the message count ``n`` and how message lengths are drawn
(``dist``: ``fixed`` at ``len`` bytes, ``uniform`` on 0..``len``, ``lognormal`` with median
``len``, sigma 1.5 and cap ``cap``).  Messages are uniform random bytes, packed back to
back, so a ragged batch's messages start at any byte.

Outputs are digests (bytes); ``exact`` gives them from hashlib where that is quick.
"""
from __future__ import annotations

import hashlib
import math
from statistics import NormalDist

import numpy as np
import torch

from paper_2407_09333_amd import DIGEST_SIZE, hb, workloads

ALGOS = ("md5", "sha1", "sm3")
# 32-bit integer operations per 64-byte block that the compressions cannot do without
# (three-input logic, rotates and three-term sums as one each)
BLOCK_OPS = {"md5": 324, "sha1": 613, "sm3": 1348}
SIGMA = 1.5            # of the log-normal lengths
KIB, MIB = 1 << 10, 1 << 20


def listed() -> list[dict]:
    return [
        # one call on a few thousand short records (keys, identifiers): one padded block each,
        # bound by the call and launch
        {"name": "md5_short", "op": "fixed", "algo": "md5", "n": 4096, "dist": "fixed", "len": 55, "cap": 0},
        # tree nodes: two 32-byte child digests hashed into one, a level of an odd width
        {"name": "sm3_nodes", "op": "fixed", "algo": "sm3", "n": 300_007, "dist": "fixed", "len": 64, "cap": 0},
        # memory or storage pages hashed for deduplication, a batch that does not fill the chip
        {"name": "sha1_pages", "op": "fixed", "algo": "sha1", "n": 20_011, "dist": "fixed", "len": 4096, "cap": 0},
        # the benchmark's headline step: the same 2^20 x 1 KiB buffer through all three algorithms
        {"name": "headline_step", "op": "fixed_step", "algo": "all", "n": 1 << 20, "dist": "fixed", "len": 1024, "cap": 0},
        # records of very different lengths in one plain call
        {"name": "sha1_ragged", "op": "plain", "algo": "sha1", "n": 200_003, "dist": "lognormal", "len": 256, "cap": 64 * KIB},
        # per-message algorithms in one plain call
        {"name": "mixed_plain", "op": "plain", "algo": "mixed", "n": 50_021, "dist": "lognormal", "len": 512, "cap": 64 * KIB},
        # one serving request's messages, hashed by a caller that cannot allocate
        {"name": "sm3_request", "op": "noalloc", "algo": "sm3", "n": 2_503, "dist": "lognormal", "len": 256, "cap": 64 * KIB},
        # the batched form on uneven lengths, resident in HBM
        {"name": "sm3_uneven", "op": "plan", "algo": "sm3", "n": 1 << 22, "dist": "uniform", "len": 4096, "cap": 0},
        # the batched form on a large mixed batch with messages up to 1 MiB (about 8 GiB)
        {"name": "mixed_8gib", "op": "plan", "algo": "mixed", "n": 5_450_000, "dist": "lognormal", "len": 512, "cap": MIB},
        # a tenth of the nine-digit decimal strings, generated on the device
        {"name": "sha1_digits", "op": "digits", "algo": "sha1", "n": 100_000_000, "dist": "fixed", "len": 9, "cap": 0},
        # messages that arrive in four pieces: init, three updates, final
        {"name": "sm3_stream", "op": "stream", "algo": "sm3", "n": 262_147, "dist": "fixed", "len": 1024, "cap": 0},
        # a batch in pageable host memory, digests back on the host
        {"name": "sm3_host", "op": "host", "algo": "sm3", "n": 16_384, "dist": "fixed", "len": 1024, "cap": 0},
    ]


def _logint(rng, lo: int, hi: int) -> int:
    """Log-uniform integer on [lo, hi], odd more often than not."""
    v = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    if rng.random() < 0.7:
        v |= 1
    return max(lo, min(hi, v))


def draw(rng) -> dict:
    op = rng.choice(["fixed", "fixed", "plain", "plain", "noalloc", "plan", "plan", "digits", "stream", "host"])
    algo = rng.choice(ALGOS)
    if op == "digits":
        return {"op": op, "algo": algo, "n": _logint(rng, 1_000, 100_000_000), "dist": "fixed", "len": 9, "cap": 0}
    if op == "fixed":
        length = _logint(rng, 1, 64 * KIB)
        if rng.random() < 0.5:  # whole dwords, as records usually are
            length = max(4, length & ~3)
        n = _logint(rng, 64, min(1 << 20, max(64, (1 << 30) // length)))
        return {"op": op, "algo": algo, "n": n, "dist": "fixed", "len": length, "cap": 0}
    if op == "stream":  # four pieces, the first three of whole blocks
        length = 256 * _logint(rng, 1, 16)
        return {"op": op, "algo": algo, "n": _logint(rng, 64, min(1 << 20, (1 << 30) // length)), "dist": "fixed",
                "len": length, "cap": 0}
    if op == "host":
        length = _logint(rng, 16, 8 * KIB)
        return {"op": op, "algo": algo, "n": _logint(rng, 16, min(1 << 17, (1 << 26) // length)), "dist": "uniform",
                "len": length, "cap": 0}
    if rng.random() < 0.5:
        algo = "mixed"
    top = {"plain": 1 << 18, "noalloc": 1 << 17, "plan": 1 << 21}[op]
    n = _logint(rng, 64, top)
    if rng.random() < 0.5:
        return {"op": op, "algo": algo, "n": n, "dist": "uniform", "len": _logint(rng, 16, 4096), "cap": 0}
    return {"op": op, "algo": algo, "n": n, "dist": "lognormal", "len": _logint(rng, 32, 1024),
            "cap": rng.choice([4 * KIB, 64 * KIB])}


def _lengths(case: dict, rng) -> np.ndarray:
    if case["dist"] == "fixed":
        return np.full(case["n"], case["len"], np.uint64)
    if case["dist"] == "uniform":
        return rng.integers(0, case["len"] + 1, size=case["n"], dtype=np.uint64)
    return workloads.lognormal_lengths(rng, case["n"], float(case["len"]), SIGMA, case["cap"])


def _host_inputs(case: dict, seed: int):
    """Lengths, offsets and algorithm ids (None for one algorithm), from the seed."""
    rng = np.random.Generator(np.random.PCG64(seed))
    lens = _lengths(case, rng)
    algos = rng.integers(0, 3, size=case["n"], dtype=np.uint8) if case["algo"] == "mixed" else None
    return lens, workloads.packed(lens), algos


def prepare(case: dict, seed: int) -> dict:
    st = {"case": case}
    op = case["op"]
    if op == "digits":
        st["start"] = (seed * 7_919_003) % (1_000_000_000 - case["n"] + 1)
        return st
    if op in ("fixed", "fixed_step"):
        st["msgs"] = workloads.device_random_bytes(case["n"] * case["len"], seed)
        return st
    if op == "stream":
        piece, n = case["len"] // 4, case["n"]
        st["msgs"] = workloads.device_random_bytes(n * case["len"], seed)
        first = torch.arange(n, dtype=torch.int64, device="cuda") * case["len"]
        st["offs"] = [first + k * piece for k in range(4)]
        st["lens"] = torch.full((n,), piece, dtype=torch.int64, device="cuda")
        return st
    lens, offs, algos = _host_inputs(case, seed)
    nbytes = int(lens.sum())
    if op == "host":
        st.update(msgs=workloads.host_random_bytes(nbytes, seed), offs=offs, lens=lens)
        return st
    st["msgs"] = workloads.device_random_bytes(max(nbytes, 4), seed)
    st["offs"] = torch.from_numpy(offs.astype(np.int64)).cuda()
    st["lens"] = torch.from_numpy(lens.astype(np.int64)).cuda()
    st["algos"] = torch.from_numpy(algos).cuda() if algos is not None else None
    if op == "plan":
        st["plan"] = hb.Plan(case["n"])
    return st


def run(st: dict):
    case = st["case"]
    op, algo = case["op"], case["algo"]
    if op == "fixed":
        return hb.hash_batch_fixed(algo, st["msgs"], case["n"], case["len"])
    if op == "fixed_step":
        return [hb.hash_batch_fixed(a, st["msgs"], case["n"], case["len"]) for a in ALGOS]
    if op == "digits":
        return hb.hash_digits9(algo, st["start"], case["n"])
    if op == "stream":
        states = hb.hash_init(algo, case["n"])
        for k in range(3):
            hb.hash_update(algo, states, st["msgs"], st["offs"][k], st["lens"])
        return hb.hash_final(algo, states, st["msgs"], st["offs"][3], st["lens"])
    if op == "host":
        return hb.hash_batch_host(st["msgs"], st["offs"], st["lens"], algo=algo)
    one = None if algo == "mixed" else algo
    if op == "plan":
        return st["plan"].run(st["msgs"], st["offs"], st["lens"], algo=one, algos=st["algos"])
    if op == "noalloc":
        return hb.hash_batch_bucketed_noalloc(st["msgs"], st["offs"], st["lens"], algo=one, algos=st["algos"])
    if one is None:
        return hb.hash_batch_mixed(st["algos"], st["msgs"], st["offs"], st["lens"])
    return hb.hash_batch(one, st["msgs"], st["offs"], st["lens"])


def _mean_length(case: dict) -> float:
    if case["dist"] == "fixed":
        return float(case["len"])
    if case["dist"] == "uniform":
        return case["len"] / 2.0
    mu, nd = math.log(case["len"]), NormalDist()
    top = math.log(case["cap"])
    return (math.exp(mu + SIGMA * SIGMA / 2) * nd.cdf((top - mu - SIGMA * SIGMA) / SIGMA)
            + case["cap"] * (1 - nd.cdf((top - mu) / SIGMA)))


def work(case: dict) -> dict:
    """Bytes: each message read once, each digest written once, 16 bytes of offset and length
    per message where the call takes them.  Operations: 32-bit integer ones (see BLOCK_OPS)."""
    n, mean, algo = case["n"], _mean_length(case), case["algo"]
    names = ALGOS if algo in ("all", "mixed") else (algo,)
    blocks = (case["len"] + 8) // 64 + 1 if case["dist"] == "fixed" else (mean + 8) / 64 + 0.5
    ops = n * blocks * sum(BLOCK_OPS[a] for a in names)
    digest = sum(DIGEST_SIZE[hb.ALGO_IDS[a]] for a in names)
    data = n * mean
    if algo == "all":
        data *= len(names)  # one call per algorithm
    elif algo == "mixed":
        ops /= len(names)
        digest = 33         # a 32-byte slot and the id
    if case["op"] == "digits":
        data = 0            # generated on the device
    elif case["op"] not in ("fixed", "fixed_step"):
        digest += 16
    return {"bytes": data + n * digest, "flops": ops}


def _hash(name: str, data) -> bytes:
    return hashlib.new(name, data).digest()


def exact(case: dict, seed: int):
    """The digests by hashlib; None where that would take long."""
    n, op = case["n"], case["op"]
    if n > 400_000 or n * _mean_length(case) > 192 * MIB:
        return None
    if op == "digits":
        start = (seed * 7_919_003) % (1_000_000_000 - n + 1)
        texts = (b"%09d" % i for i in range(start, start + n))
        out = b"".join(_hash(case["algo"], t) for t in texts)
        return torch.from_numpy(np.frombuffer(out, np.uint8).reshape(n, -1).copy())
    lens, offs, algos = _host_inputs(case, seed)
    nbytes = int(lens.sum())
    if op == "host":
        data = workloads.host_random_bytes(nbytes, seed)
    else:
        data = workloads.device_random_bytes(max(nbytes, 4), seed).cpu().numpy()
    view = memoryview(data)
    names = [case["algo"]] * n if algos is None else [ALGOS[a] for a in algos]
    stride = 32 if algos is not None else DIGEST_SIZE[hb.ALGO_IDS[case["algo"]]]
    ends = (offs + lens).tolist()
    out = b"".join(_hash(a, view[o:e]).ljust(stride, b"\0") for a, o, e in zip(names, offs.tolist(), ends))
    res = np.frombuffer(out, np.uint8).reshape(n, stride).copy()
    return res if op == "host" else torch.from_numpy(res)
