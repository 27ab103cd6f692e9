"""The plan's bucketed pipeline, asked for by a launch choice (a plan without one runs the
tiled launch): graph replay, the long-chain path on a side stream, in one launch and in a
graph, scratch regions past the saturated sort key, and batches on both sides of one wave
per SIMD.  Every digest bit-exact against the oracle."""
import numpy as np
import pytest

import oracle
from paper_2407_09333_amd import workloads
from tests.gpu_util import assert_same, check_guard, guarded_out
from tests.test_gpu_plan import _batch_mixed_with_long, _saturated_long_batch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hb():
    import torch

    assert torch.cuda.is_available()
    from paper_2407_09333_amd import hb as _hb

    return _hb


def pipeline(hb, n, flags):
    plan = hb.Plan(n, flags=flags)
    plan.set_config(waves_per_cu=16, msgs_per_lane=1, variant=0)
    return plan


def run_guarded(plan, n, stride, *args, **kw):
    buf, out = guarded_out(n, stride)
    plan.run(*args, out=out, **kw)
    check_guard(buf, n, stride)
    return out.cpu().numpy()


def test_graph_replays_with_changing_inputs(hb):
    """Captured pipelines replayed over batches of different sizes, on both sides of one wave
    per SIMD, with eager torch work and synchronisations in between."""
    import torch

    plan_g, plan_e = pipeline(hb, 100_000, hb.PLAN_GRAPH), pipeline(hb, 100_000, 0)
    for rep, (n, seed) in enumerate([(40_000, 1), (1_000, 2), (100_000, 3), (7, 4), (90_000, 5), (40_000, 1), (100_000, 6)]):
        print(f"case pipeline replay {rep} n={n}", flush=True)
        b = workloads.mixed_batch(n * 2400 + 100_000, seed=seed, cap=1 << 14)
        assert b.n >= n
        offs, lens, al = b.offsets[:n], b.lengths[:n], b.algos[:n]
        x = torch.randn(1000, device="cuda")
        (x * 2).sum().item()  # eager work between replays
        got = plan_g.run(b.messages, offs, lens, algos=al)
        torch.cuda.synchronize()
        ref = plan_e.run(b.messages, offs, lens, algos=al)
        want = oracle.hash_batch(al, b.messages, offs, lens)
        assert_same(got.cpu().numpy(), want, f"replay {rep}")
        assert_same(ref.cpu().numpy(), want, f"eager {rep}")
    plan_g.close()
    plan_e.close()


@pytest.mark.parametrize("flags", [1, 0], ids=["graph", "eager"])
def test_single_and_mixed(hb, flags):
    for algo in (0, 1, 2):
        print(f"case pipeline single algo={algo} flags={flags}", flush=True)
        b = workloads.uniform_lengths_batch(algo, 20_000, 4096, seed=13)
        plan = pipeline(hb, 32_768, flags)
        ds = oracle.DIGEST_SIZE[algo]
        got = run_guarded(plan, b.n, ds, b.messages, b.offsets, b.lengths, algo=algo)
        assert_same(got, oracle.hash_batch(algo, b.messages, b.offsets, b.lengths), "pipeline single")
        plan.close()
    msgs, offs, lens, algos = _batch_mixed_with_long()
    al = algos.copy()
    al[::101] = 200  # unknown: an all-zero slot
    print(f"case pipeline mixed flags={flags}", flush=True)
    plan = pipeline(hb, offs.size, flags)
    want = oracle.hash_batch(algos, msgs, offs, lens)
    want[::101] = 0
    assert_same(run_guarded(plan, offs.size, 32, msgs, offs, lens, algos=al), want, "pipeline mixed")
    plan.close()


@pytest.mark.parametrize("scratch_mb,min_blocks", [("1", "256"), ("512", "2"), ("1024", "16")])
def test_long_chain_path(hb, monkeypatch, scratch_mb, min_blocks):
    """Messages above the block threshold as rounds-only chains from precomputed schedule
    words, those that the scratch cannot hold as direct chains; beside the bulk on a side
    stream, or in one launch with it; eager and in a graph, two runs each."""
    monkeypatch.setenv("HB_LONG_SCRATCH_MB", scratch_mb)
    monkeypatch.setenv("HB_LONG_MIN_BLOCKS", min_blocks)
    rng = np.random.default_rng(int(min_blocks))
    n = 3000
    lens = rng.integers(0, 40_000, size=n).astype(np.uint64)
    lens[:40] = rng.integers(100_000, 300_000, size=40)
    lens[40:50] = [0, 1, 55, 56, 63, 64, 119, 120, 16_384, 16_383]
    offs = workloads.packed(lens)
    msgs = workloads.host_random_bytes(int(lens.sum()), seed=int(min_blocks) + 1)
    algos = rng.integers(0, 3, size=n).astype(np.uint8)
    want = oracle.hash_batch(algos, msgs, offs, lens)
    for flags in (hb.PLAN_GRAPH, 0, hb.PLAN_GRAPH | hb.PLAN_LONG_INLINE, hb.PLAN_LONG_INLINE, hb.PLAN_NO_LONG):
        print(f"case pipeline long path scratch={scratch_mb} min_blocks={min_blocks} flags={flags}", flush=True)
        plan = pipeline(hb, n, flags)
        for _ in range(2):
            assert_same(run_guarded(plan, n, 32, msgs, offs, lens, algos=algos), want, f"long path flags={flags}")
        plan.close()


@pytest.mark.parametrize("scratch_mb", ["1024", "2048", "4096"])
def test_long_chains_past_key_saturation(hb, monkeypatch, scratch_mb):
    """Many messages of one algorithm above the saturated sort key: a long-chain wave's scratch
    region must hold its longest lane.  1 GiB holds no such wave (direct chains), 2 GiB the
    first of SM3's and 4 GiB both."""
    monkeypatch.setenv("HB_LONG_SCRATCH_MB", scratch_mb)
    msgs, offs, lens, algos = _saturated_long_batch()
    want = oracle.hash_batch(algos, msgs, offs, lens)
    for flags in (hb.PLAN_GRAPH, hb.PLAN_LONG_INLINE):
        print(f"case pipeline saturated scratch={scratch_mb} flags={flags}", flush=True)
        plan = pipeline(hb, lens.size, flags)
        assert_same(run_guarded(plan, lens.size, 32, msgs, offs, lens, algos=algos), want, f"saturated flags={flags}")
        plan.close()
    sm3 = np.nonzero(algos == 2)[0]  # the segment holds saturated keys first
    plan = pipeline(hb, sm3.size, hb.PLAN_GRAPH)
    assert_same(run_guarded(plan, sm3.size, 32, msgs, offs[sm3], lens[sm3], algo=2), want[sm3, :32], "saturated sm3 only")
    plan.close()


@pytest.mark.parametrize("variant", range(5))
def test_both_sides_of_one_wave_per_simd(hb, variant):
    """As many items as SIMDs and one more (messages per lane 1 and 2), every load scheme; the
    same without sorting."""
    simds = 4 * hb.device_info()["cu_count"]
    for n, mpl in ((64 * simds, 1), (64 * simds + 1, 1), (128 * simds, 2), (128 * simds + 1, 2)):
        for algo in (0, 1, 2):
            print(f"case pipeline few variant={variant} n={n} mpl={mpl} algo={algo}", flush=True)
            b = workloads.uniform_lengths_batch(algo, n, 300, seed=n % 1000 + algo)
            want = oracle.hash_batch(algo, b.messages, b.offsets, b.lengths)
            for flags in (0, hb.PLAN_NO_SORT):
                plan = hb.Plan(n, flags=flags)
                plan.set_config(waves_per_cu=16, msgs_per_lane=mpl, variant=variant)
                got = run_guarded(plan, n, oracle.DIGEST_SIZE[algo], b.messages, b.offsets, b.lengths, algo=algo)
                assert_same(got, want, f"few {variant} {flags}")
                plan.close()


def test_the_form_that_runs_is_reported(hb):
    """A plan says whether it runs the tiled launch; launch choices and unsorted plans have it
    run the pipeline; an autotuned one settles it with its first run, after which a plan set up
    as it reports has the same form."""
    b = workloads.uniform_lengths_batch(2, 3_000, 2048, seed=81)
    want = oracle.hash_batch(2, b.messages, b.offsets, b.lengths)
    plan = hb.Plan(b.n)
    assert plan.tiled()
    plan.set_config(waves_per_cu=8)
    assert not plan.tiled()
    plan.close()
    plan = hb.Plan(b.n, flags=hb.PLAN_NO_SORT)
    assert not plan.tiled()
    plan.close()
    plan = hb.Plan(b.n, flags=hb.PLAN_AUTOTUNE)
    assert_same(plan.run(b.messages, b.offsets, b.lengths, algo=2).cpu().numpy(), want, "autotuned")
    twin = hb.Plan(b.n, flags=0)
    if not plan.tiled():
        twin.set_config(**plan.config())
    assert twin.tiled() == plan.tiled()
    assert_same(twin.run(b.messages, b.offsets, b.lengths, algo=2).cpu().numpy(), want, "twin")
    assert twin.kernel_ms() > 0
    plan.close()
    twin.close()
