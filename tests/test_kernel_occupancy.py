"""Host check (not a GPU test): waves per SIMD that the compiled mixed map kernel of
visit lists allows.  Three, whatever its register count: lists of some 800 blocks
are dealt unevenly over the compute units, and the fullest one decides."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_visit_map_waves(tmp_path):
    hipcc = shutil.which(os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"))
    if not hipcc:
        pytest.skip("no hipcc")
    from paper_2507_00294_amd import build

    out = tmp_path / "visits.s"
    subprocess.run([hipcc, *build.FLAGS, "-S", "--offload-device-only",
                    os.path.join(ROOT, "paper_2507_00294_amd/csrc/dd_visits.hip"), "-o", str(out)],
                   check=True, capture_output=True)
    text = out.read_text()
    body = text[re.search(r"^_ZN2dd\S*k_visit_map\S*:", text, re.M).start():]
    assert re.search(r"; Occupancy: (\d+)", body).group(1) == "3"
