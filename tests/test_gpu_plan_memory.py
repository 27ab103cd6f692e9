"""What plans hold on the device: a plan that runs the tiled launch holds no schedule scratch.
The scratch is 1 GiB; streams and the runtime's own allocations are counted with it, so the
bounds lie halfway between one scratch more and one fewer."""
import pytest

pytestmark = pytest.mark.gpu

GIB = 1 << 30


@pytest.fixture(scope="module")
def hb():
    import torch

    assert torch.cuda.is_available()
    from paper_2407_09333_amd import hb as _hb

    return _hb


def free_bytes():
    import torch

    torch.cuda.synchronize()
    return torch.cuda.mem_get_info()[0]


def test_schedule_scratch_comes_with_the_pipeline(hb):
    before = free_bytes()
    plan = hb.Plan(1000)
    assert before - free_bytes() < GIB // 2
    plan.set_config(waves_per_cu=16, msgs_per_lane=1, variant=0)
    assert before - free_bytes() >= GIB // 2
    plan.set_config(waves_per_cu=8)  # no second one
    assert before - free_bytes() < GIB + GIB // 2
    plan.close()
    assert before - free_bytes() < GIB // 2


@pytest.mark.parametrize("env,flags", [(None, 2), ("8", 0)], ids=["autotune", "waves_per_cu"])
def test_plans_that_may_take_the_pipeline_have_it_from_the_start(hb, monkeypatch, env, flags):
    if env:
        monkeypatch.setenv("HB_WAVES_PER_CU", env)
    before = free_bytes()
    plan = hb.Plan(1000, flags=flags)
    assert before - free_bytes() >= GIB // 2
    plan.close()


def test_scratch_that_cannot_be_allocated(hb, monkeypatch):
    """set_config reports it and leaves the plan as it was; a smaller scratch then works."""
    monkeypatch.setenv("HB_LONG_SCRATCH_MB", str(1 << 20))  # 1 TiB
    plan = hb.Plan(1000)
    with pytest.raises(hb.HBError) as e:
        plan.set_config(waves_per_cu=8, msgs_per_lane=2, variant=1)
    assert e.value.status == hb.HB_ENOMEM
    assert plan.config() == {"waves_per_cu": 16, "msgs_per_lane": 1, "variant": 0}
    plan.close()


def test_server_holds_no_schedule_scratch(hb):
    before = free_bytes()
    srv = hb.Server(hbm_budget_bytes=64 << 20, max_slots=8)
    assert before - free_bytes() < GIB // 2
    srv.close()
