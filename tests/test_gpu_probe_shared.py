"""The issue-rate probe's kinds for the shared-SIMD order: with four waves on a SIMD the runs at
two priorities issue faster than the same instructions mixed, and the shared form of each
compression faster than the compiler's order; neither beats the two places a SIMD has."""
import pytest

from tests.test_gpu_probe import OPS_BY_RATE

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hb():
    import torch

    assert torch.cuda.is_available()
    from paper_2407_09333_amd import hb as _hb

    return _hb


def test_shared_order_issues_faster(hb):
    print("case probe shared", flush=True)
    mixed = hb.probe_valu("mix_bitop3_alignbit_3_1", 4)[0]
    runs = hb.probe_valu("mix_bitop3_alignbit_3_1_runs", 4)[0]
    assert 1.95 < runs < 0.9 * mixed  # 2.0: both places busy
    for a in OPS_BY_RATE:
        alone, shared = hb.probe_valu(a, 4)[0], hb.probe_valu(a + "_shared", 4)[0]
        # a SIMD's two places finish at most one instruction each in four cycles, and the fewest
        # instructions that a block can take are the counted ones
        assert 2 * sum(OPS_BY_RATE[a]) * 0.95 < shared < alone, a
