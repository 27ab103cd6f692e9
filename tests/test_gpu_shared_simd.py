"""Launches on both sides of one wave per SIMD: up to there a lane runs the compression with
the fewest instructions, past it the one ordered for SIMDs that several waves share.  Every
digest bit-exact against the oracle, through each entry point that takes either."""
import numpy as np
import pytest

import oracle
from paper_2407_09333_amd import workloads
from tests.gpu_util import assert_same

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hb():
    import torch

    assert torch.cuda.is_available()
    from paper_2407_09333_amd import hb as _hb

    return _hb


@pytest.mark.parametrize("algo", [0, 1, 2])
@pytest.mark.parametrize("extra", [0, 1])
def test_both_sides_of_one_wave_per_simd(hb, algo, extra):
    n = hb.device_info()["cu_count"] * 4 * 64 + extra
    print(f"case shared simd algo={algo} n={n}", flush=True)
    for L in (61, 128, 196):  # per lane; staged through LDS with and without a padding-only last block
        b = workloads.fixed_batch(algo, n, L, seed=700 + L)
        got = hb.hash_batch_fixed(algo, b.messages, n, L).cpu().numpy()
        assert_same(got, oracle.hash_batch(algo, b.messages, b.offsets, b.lengths), f"fixed {L}")
    b = workloads.uniform_lengths_batch(algo, n, 300, seed=701)
    want = oracle.hash_batch(algo, b.messages, b.offsets, b.lengths)
    assert_same(hb.hash_batch(algo, b.messages, b.offsets, b.lengths).cpu().numpy(), want, "packed")
    plan = hb.Plan(n)
    assert_same(plan.run(b.messages, b.offsets, b.lengths, algo=algo).cpu().numpy(), want, "plan")
    plan.close()
    b = workloads.fixed_batch(algo, n, 192 + 7, seed=702)
    offs = b.offsets.astype(np.int64)
    states = hb.hash_init(algo, n)
    hb.hash_update(algo, states, b.messages, offs, np.full(n, 192, np.int64))
    got = hb.hash_final(algo, states, b.messages, offs + 192, np.full(n, 7, np.int64)).cpu().numpy()
    assert_same(got, oracle.hash_batch(algo, b.messages, b.offsets, b.lengths), "incremental")
    b = workloads.digits9_batch(n, start=5)
    assert_same(hb.hash_digits9(algo, 5, n).cpu().numpy(),
                oracle.hash_batch(algo, b.messages, b.offsets, b.lengths), "digits")
