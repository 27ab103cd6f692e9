"""Register and LDS budgets of the kernels for shared SIMDs and of the tiled launches, read from
the gfx950 code objects' metadata: no vector spills or private memory, and the occupancy that
each is built for.  A change that pushed a kernel past its budget would slow it silently."""
import re
import shutil
import subprocess
from pathlib import Path

import pytest

ROOT = Path(__file__).resolve().parent.parent
CSRC = ROOT / "paper_2407_09333_amd" / "csrc"
HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"

# kernel, as demangled up to its arguments -> largest VGPR count (512 per SIMD lane in granules
# of 8: 96 leave five waves per SIMD, 128 four, 168 three) and largest LDS size (160 KiB a CU)
BUDGETS = {
    "hb_kernels.hip": {
        **{f"k_plain_lds_pad<{a}>": (96, 32768) for a in range(3)},  # five waves, as the LDS holds
        "k_plain_lds<2>": (96, 32768),
    },
    "hb_ragged.hip": {
        # four workgroups of four waves to a CU: one chain wave to each SIMD
        **{f"k_ragged<{a}, {many}, {per}>": (128, 40960)
           for a in range(3) for many, per in (("false", 1), ("true", 1), ("true", 2), ("true", 8))},
        "k_ragged_mixed<true, 2>": (128, 40960),
        "k_ragged_mixed<true, 8>": (128, 40960),
        "k_ragged_mixed<false, 2>": (168, 40960),
        **{f"k_long_tiles<{a}>": (128, 40960) for a in (-1, 0, 1, 2)},
        # one workgroup to a CU
        **{f"k_fixed_chain<{a}>": (128, 160 * 1024) for a in range(3)},
    },
}


def kernels(source):
    if not Path(HIPCC).exists():
        pytest.skip("hipcc not available")
    cmd = [HIPCC, "-O3", "-std=c++17", f"-I{ROOT / 'include'}", "--offload-arch=gfx950", "--offload-device-only",
           "-S", "-x", "hip", str(CSRC / source), "-o", "-", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stderr[-2000:]
    found = {}
    for block in re.split(r"\n  - \.", r.stdout)[1:]:  # one kernel per item of .amdhsa.kernels
        m = re.search(r"^    \.name:\s+(\S+)", block, re.M)  # the kernel's own fields: four spaces in
        if m:
            found[m.group(1)] = {k: int(v) for k, v in re.findall(
                r"^    \.(vgpr_count|vgpr_spill_count|private_segment_fixed_size|group_segment_fixed_size):\s+(\d+)", block, re.M)}
    names = subprocess.run(["c++filt"], input="\n".join(found), capture_output=True, text=True).stdout.split("\n")
    short = [re.sub(r"^void ", "", n).replace("(anonymous namespace)::", "").removeprefix("hb::").split("(")[0] for n in names]
    return dict(zip(short, found.values()))


@pytest.mark.parametrize("source", BUDGETS)
def test_budgets(source):
    found = kernels(source)
    for name, (vgprs, lds) in BUDGETS[source].items():
        assert name in found, (name, sorted(found))
        assert found[name]["vgpr_count"] <= vgprs, (name, found[name])
        assert found[name]["group_segment_fixed_size"] <= lds, (name, found[name])
    for name, k in found.items():
        assert k.get("vgpr_spill_count", 0) == 0 and k.get("private_segment_fixed_size", 0) == 0, (name, k)
