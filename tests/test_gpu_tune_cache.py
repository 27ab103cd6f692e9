"""The autotuner's cache: a choice is kept for the plans and batches it was made for, and lines
written before the cache said which those are give only the pipeline's choices."""
import os
import subprocess
import sys
from pathlib import Path

import pytest

pytestmark = pytest.mark.gpu

ROOT = Path(__file__).resolve().parent.parent

# autotuned plans over one batch, each digest checked; prints each plan's choice and form
CHILD = """
import sys
import torch
import oracle
from paper_2407_09333_amd import hb, workloads
b = workloads.uniform_lengths_batch(2, 20_000, 2000, seed=5)
want = oracle.hash_batch(2, b.messages, b.offsets, b.lengths)
for flags in map(int, sys.argv[1:]):
    plan = hb.Plan(b.n, flags=flags | hb.PLAN_AUTOTUNE)
    for _ in range(2):
        got = plan.run(b.messages, b.offsets, b.lengths, algo=2).cpu().numpy()
        assert (got == want).all(), flags
    c = plan.config()
    print(c["waves_per_cu"], c["msgs_per_lane"], c["variant"], int(plan.tiled()))
    plan.close()
"""


def tune(cache, *flags):
    print(f"case tune cache flags={flags}", flush=True)
    env = dict(os.environ, HB_TUNE_CACHE=str(cache), PYTHONPATH=str(ROOT))
    r = subprocess.run([sys.executable, "-c", CHILD, *map(str, flags)], cwd=ROOT, env=env, capture_output=True,
                       text=True, timeout=100)
    assert r.returncode == 0, r.stderr[-2000:]
    lines = [ln.split() for ln in cache.read_text().splitlines()]
    return [list(map(int, ln.split())) for ln in r.stdout.splitlines()], lines


def test_choices_are_kept_by_form(tmp_path):
    cache = tmp_path / "tune.txt"
    picked, lines = tune(cache, 0, 8, 0)  # sorted with and without the long-chain path
    assert len(lines) == 2 and all(len(ln) == 9 for ln in lines), lines
    assert lines[0][:4] == lines[1][:4] and lines[0][8] != lines[1][8]
    assert picked[2] == picked[0]
    kept = {tuple(map(int, ln[4:8])) for ln in lines}
    assert {tuple(p) for p in picked} <= kept
    again, same = tune(cache, 0, 8)  # another process takes both from the file
    assert again == picked[:2] and same == lines


@pytest.mark.parametrize("numbers", [7, 8])
def test_lines_without_a_form(tmp_path, numbers):
    """The pipeline's choices of such a line are taken over, timed against the tiled launch and
    kept with a form beside it."""
    cache = tmp_path / "tune.txt"
    _, lines = tune(cache, 0)
    old = " ".join(lines[0][:4] + ["8", "2", "3", "0"][: numbers - 4])
    cache.write_text(old + "\n")
    picked, lines = tune(cache, 0)
    assert picked[0][:3] == [8, 2, 3]
    new = [ln for ln in lines if len(ln) == 9]
    assert len(lines) == 2 and len(new) == 1 and list(map(int, new[0][4:8])) == picked[0], lines
