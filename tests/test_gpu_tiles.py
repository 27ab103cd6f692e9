"""Packed batches where the rule for their tiles changes (hb_plan_rules.hpp): every digest
bit-exact against the oracle, with no write outside the digest buffer."""
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


def check_batch(hb, lens, seed, what, mixed=True):
    """Each algorithm on its own and (mixed) all three, through hash_batch's tiles."""
    n = lens.size
    lens = lens.astype(np.uint64)
    offs = workloads.packed(lens)
    msgs = workloads.host_random_bytes(int(lens.sum()) + 1, seed=seed)
    for algo in (0, 1, 2):
        print(f"case {what} n={n} algo={algo}", flush=True)
        ds = oracle.DIGEST_SIZE[algo]
        buf, out = guarded_out(n, ds)
        hb.hash_batch(algo, msgs, offs, lens, out=out)
        check_guard(buf, n, ds)
        assert_same(out.cpu().numpy(), oracle.hash_batch(algo, msgs, offs, lens), f"{what} {algo}")
    if mixed:
        print(f"case {what} n={n} mixed", flush=True)
        algos = np.random.default_rng(seed).integers(0, 3, n).astype(np.uint8)
        buf, out = guarded_out(n, 32)
        hb.hash_batch_mixed(algos, msgs, offs, lens, out=out)
        check_guard(buf, n, 32)
        assert_same(out.cpu().numpy(), oracle.hash_batch(algos, msgs, offs, lens), f"{what} mixed")


@pytest.mark.parametrize("length", [4100, 200])
@pytest.mark.parametrize("per_cu", [1, 8, 32])
@pytest.mark.parametrize("extra", [-1, 0, 1])
def test_few_alike_messages(hb, length, per_cu, extra):
    """Messages of one length, on both sides of the counts where every one of a tile runs in
    its chain pair (32 to a CU, eight of MD5; 64 to three CUs where algorithms are mixed)."""
    cus = hb.device_info()["cu_count"]
    check_batch(hb, np.full(per_cu * cus + extra, length), 3, "few alike", mixed=False)
    n = 2 * per_cu * (cus // 3) + extra
    offs = np.arange(n, dtype=np.uint64) * np.uint64(length)
    msgs = workloads.host_random_bytes(n * length, seed=4)
    algos = np.random.default_rng(5).integers(0, 3, n).astype(np.uint8)
    lens = np.full(n, length, np.uint64)
    got = hb.hash_batch_mixed(algos, msgs, offs, lens).cpu().numpy()
    assert_same(got, oracle.hash_batch(algos, msgs, offs, lens), "few alike mixed")


@pytest.mark.parametrize("per_cu", [1024, 1025, 2048, 2049, 2300])
def test_messages_in_index_order(hb, per_cu):
    """Messages of one block count, hashed in index order: tiles of one message a thread, two
    and more, and tiles that are no multiple of 256."""
    n = per_cu * hb.device_info()["cu_count"] + 7
    check_batch(hb, 16 + np.arange(n) % 7, 6, "index order", mixed=False)


@pytest.mark.parametrize("longest", [63, 64])
@pytest.mark.parametrize("per_cu", [2300, 4096, 6200, 8192])
def test_short_messages_sorted_512_at_a_time(hb, per_cu, longest):
    """Short messages in tiles of one to four times 512, and a little more, the longest on both
    sides of the last block count that is sorted so."""
    n = per_cu * hb.device_info()["cu_count"] - 5
    rng = np.random.default_rng(longest)
    lens = rng.integers(0, 150, n)
    lens[rng.choice(n, 3 * n // 2000, replace=False)] = 64 * longest - 9   # in most tiles
    check_batch(hb, lens, 7, "short sorted", mixed=per_cu == 2300)


def test_mixed_batches_of_one_wave_per_simd(hb):
    """Mixed batches on both sides of one wave per SIMD: the workgroups have about a third of a
    tile each."""
    cus = hb.device_info()["cu_count"]
    for n in (64 * cus, 128 * cus + 1, 226 * cus, 226 * cus + 1, 256 * cus):
        print(f"case mixed few n={n}", flush=True)
        rng = np.random.default_rng(n)
        lens = rng.integers(0, 700, n).astype(np.uint64)
        algos = rng.integers(0, 3, n).astype(np.uint8)
        offs = workloads.packed(lens)
        msgs = workloads.host_random_bytes(int(lens.sum()) + 1, seed=8)
        got = hb.hash_batch_mixed(algos, msgs, offs, lens).cpu().numpy()
        assert_same(got, oracle.hash_batch(algos, msgs, offs, lens), f"mixed few {n}")
