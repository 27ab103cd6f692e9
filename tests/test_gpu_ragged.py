"""hash_batch / hash_batch_mixed (one launch: tiles sorted in LDS, a chain pair for a tile's
longest messages) where the tile, the chain pair's windows and the last blocks change shape.
Every digest bit-exact against the oracle, with no write outside the digest buffer."""
import numpy as np
import pytest

import oracle
from paper_2407_09333_amd import workloads
from tests.gpu_util import assert_same, check_guard, guarded_out

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hb():
    import torch

    assert torch.cuda.is_available()
    from paper_2407_09333_amd import hb as _hb

    return _hb


def lengths(kind: str, n: int) -> np.ndarray:
    rng = np.random.default_rng(n)
    if kind == "equal":            # nothing to sort
        return np.full(n, 130)
    if kind == "chains":           # every residue of the last block, 3 to about 70 blocks
        return 121 + 61 * (np.arange(n) % 73)
    if kind == "one long":         # a chain of many windows beside short messages
        x = rng.integers(0, 130, n)
        x[n // 2] = 64 * 200 + 55
        return x
    if kind == "long same":        # all of one bin, more than the chain pair takes
        return np.full(n, 64 * 65)
    return rng.integers(0, 2000, n)  # "spread"


@pytest.mark.parametrize("kind", ["equal", "chains", "one long", "long same", "spread"])
@pytest.mark.parametrize("n", [1, 2, 17, 31, 32, 33, 64, 65, 257, 5000])
def test_tiles_and_chains(hb, kind, n):
    lens = lengths(kind, n).astype(np.uint64)
    gaps = np.arange(n, dtype=np.uint64) % np.uint64(5)      # messages start at any byte
    offs = workloads.packed(lens + gaps) + np.uint64(1)
    msgs = workloads.host_random_bytes(int(offs[-1] + lens[-1]), seed=n)
    for algo in (0, 1, 2):
        print(f"case ragged kind={kind} n={n} algo={algo}", flush=True)
        stride = oracle.DIGEST_SIZE[algo] + 4
        buf, out = guarded_out(n, stride)
        hb.hash_batch(algo, msgs, offs.astype(np.int64), lens.astype(np.int64), out=out, stride=stride)
        check_guard(buf, n, stride)
        assert_same(out.cpu().numpy(), oracle.hash_batch(algo, msgs, offs, lens, out_stride=stride), f"{kind} {algo}")
    algos = np.random.default_rng(7).integers(0, 4, n).astype(np.uint8)  # 3: unknown, an all-zero slot
    buf, out = guarded_out(n, 32)
    hb.hash_batch_mixed(algos, msgs, offs.astype(np.int64), lens.astype(np.int64), out=out)
    check_guard(buf, n, 32)
    known = np.where(algos > 2, 0, algos).astype(np.uint8)
    want = oracle.hash_batch(known, msgs, offs, lens)
    want[algos > 2] = 0
    assert_same(out.cpu().numpy(), want, f"{kind} mixed")


@pytest.mark.parametrize("n", [70_001, 300_007])
def test_many_tiles(hb, n):
    """More than one workgroup per CU, and tiles past 256 messages."""
    rng = np.random.default_rng(n)
    lens = np.minimum(np.exp(rng.normal(4.0, 1.5, n)), 9000).astype(np.uint64)
    offs = workloads.packed(lens)
    msgs = workloads.host_random_bytes(int(lens.sum()) + 1, seed=3)
    for algo in (0, 1, 2):
        print(f"case many tiles n={n} algo={algo}", flush=True)
        got = hb.hash_batch(algo, msgs, offs.astype(np.int64), lens.astype(np.int64)).cpu().numpy()
        assert_same(got, oracle.hash_batch(algo, msgs, offs, lens), f"many tiles {algo}")
    algos = rng.integers(0, 3, n).astype(np.uint8)
    got = hb.hash_batch_mixed(algos, msgs, offs.astype(np.int64), lens.astype(np.int64)).cpu().numpy()
    assert_same(got, oracle.hash_batch(algos, msgs, offs, lens), "many tiles mixed")


@pytest.mark.parametrize("n", [65_536, 70_001])
@pytest.mark.parametrize("top", [64, 130, 300])
def test_short_messages(hb, n, top):
    """One message a thread, on both sides of one wave a SIMD: tiles that are not sorted
    because it would save too little, and ones that are."""
    lens = np.random.default_rng(top).integers(0, top + 1, n).astype(np.uint64)
    offs = workloads.packed(lens)
    msgs = workloads.host_random_bytes(int(lens.sum()) + 1, seed=top)
    for algo in (0, 1, 2):
        print(f"case short n={n} top={top} algo={algo}", flush=True)
        got = hb.hash_batch(algo, msgs, offs.astype(np.int64), lens.astype(np.int64)).cpu().numpy()
        assert_same(got, oracle.hash_batch(algo, msgs, offs, lens), f"short {algo}")


@pytest.mark.parametrize("blocks", [2, 3, 7, 8, 47, 48])
def test_fewest_blocks_of_a_chain(hb, blocks):
    """The longest message on each side of an algorithm's least for a chain pair."""
    lens = np.random.default_rng(blocks).integers(0, 64 * blocks - 8, 65).astype(np.uint64)
    lens[40] = 64 * blocks - 9
    offs = workloads.packed(lens)
    msgs = workloads.host_random_bytes(int(lens.sum()) + 1, seed=blocks)
    for algo in (0, 1, 2):
        got = hb.hash_batch(algo, msgs, offs.astype(np.int64), lens.astype(np.int64)).cpu().numpy()
        assert_same(got, oracle.hash_batch(algo, msgs, offs, lens), f"{blocks} blocks {algo}")


@pytest.mark.parametrize("algo", [1, 2])
@pytest.mark.parametrize("per_cu", [0, 1, 63, 64, 65, 128])
def test_few_fixed_messages(hb, algo, per_cu):
    """Fixed-length batches of few messages (chain pairs): one to 64 messages to a pair, a
    ragged last one, every residue of the last block that changes its shape, any start."""
    import torch

    cus = hb.device_info()["cu_count"]
    n = max(1, per_cu * cus - 3 if per_cu < 128 else per_cu * cus)
    for L in (120, 128, 183, 247, 256, 2047) if per_cu < 64 else (184, 2040):
        print(f"case few fixed algo={algo} n={n} L={L}", flush=True)
        b = workloads.fixed_batch(algo, n, L, seed=L)
        dev = torch.empty(b.messages.size + 1, dtype=torch.uint8, device="cuda")
        msgs = dev[1:] if L % 2 else dev[:-1]
        msgs.copy_(torch.from_numpy(b.messages))
        ds = oracle.DIGEST_SIZE[algo]
        buf, out = guarded_out(n, ds)
        hb.hash_batch_fixed(algo, msgs, n, L, out=out)
        check_guard(buf, n, ds)
        assert_same(out.cpu().numpy(), oracle.hash_batch(algo, b.messages, b.offsets, b.lengths), f"few fixed {algo} {L}")


@pytest.mark.parametrize("algo", [None, 0, 1, 2])
def test_long_messages_first(hb, monkeypatch, algo):
    """A plan whose batch has more than one round of tiles picks the longest messages out
    first: here more of them than its groups hold, some past the saturated sort key, and
    the same with the long path off."""
    monkeypatch.setenv("HB_LONG_MIN_BLOCKS", "3")
    n = 720_003 if algo is None else (1 << 21) + 1501
    rng = np.random.default_rng(90)
    lens = rng.integers(0, 100 if algo is None else 40, n)
    lens[rng.integers(0, n, 30_000)] = rng.integers(120, 1500, 30_000)
    lens[rng.integers(0, n, 40)] = rng.integers(30_000, 70_000, 40)
    lens[rng.integers(0, n, 3)] = [1_100_000, 1_060_003, 1_300_001]
    lens = lens.astype(np.uint64)
    offs = workloads.packed(lens)
    msgs = workloads.host_random_bytes(int(lens.sum()) + 1, seed=91)
    algos = rng.integers(0, 3, n).astype(np.uint8) if algo is None else None
    want = oracle.hash_batch(algo if algos is None else algos, msgs, offs, lens)
    for flags in (hb.PLAN_GRAPH, hb.PLAN_NO_LONG):
        print(f"case long first algo={algo} flags={flags}", flush=True)
        plan = hb.Plan(n, flags=flags)
        for _ in range(2):
            buf, out = guarded_out(n, want.shape[1])
            plan.run(msgs, offs, lens, algo=algo, algos=algos, out=out)
            check_guard(buf, n, want.shape[1])
            assert_same(out.cpu().numpy(), want, f"long first {algo} {flags}")
        plan.close()


@pytest.mark.parametrize("per_cu", [0, 1, 63, 64, 65])
def test_few_long_fixed_md5(hb, per_cu):
    """MD5's batches of few messages run as chain pairs from 64 blocks (4,024 bytes) on."""
    import torch

    n = max(1, per_cu * torch.cuda.get_device_properties(0).multi_processor_count - 3)
    for L in (4020, 4024, 4096, 4156):
        print(f"case few long md5 n={n} L={L}", flush=True)
        b = workloads.fixed_batch(0, n, L, seed=L)
        buf, out = guarded_out(n, 16)
        hb.hash_batch_fixed(0, torch.from_numpy(b.messages).cuda(), n, L, out=out)
        check_guard(buf, n, 16)
        assert_same(out.cpu().numpy(), oracle.hash_batch(0, b.messages, b.offsets, b.lengths), f"few long md5 {L}")
