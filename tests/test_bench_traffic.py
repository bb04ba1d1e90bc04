"""bench.py's traffic table holds what was counted: every entry is the row of its profile, and its key the kernel
sources that this profile was taken at."""
import re
import sys
from pathlib import Path

import pytest

ROOT = Path(__file__).resolve().parents[1]
sys.path.insert(0, str(ROOT))

import bench  # noqa: E402

PROFILE = {"f64": "f64", "f32": "f32", "f16": "f16", "f16+guess": "f16g"}


@pytest.mark.parametrize("key", list(bench.MEASURED_TRAFFIC), ids=lambda k: "-".join(k))
def test_entry_is_the_counted_row_of_its_profile(key):
    workload, form, sources, shape = key
    text = (ROOT / "profiles" / f"fused_step_{PROFILE[form]}_{workload}256x256x512.md").read_text()
    assert re.search(r"Kernel sources hash (\w+)", text).group(1) == sources
    assert "differ" not in re.search(r"Kernel sources hash[^\n]*", text).group(0)   # taken there, not carried over
    row = re.search(rf"^\| {re.escape(shape)} \|[^|]*\|[^|]*\| ([\d.]+) GB \|", text, re.M)
    assert row and abs(float(row.group(1)) - bench.MEASURED_TRAFFIC[key]) < 1e-9
