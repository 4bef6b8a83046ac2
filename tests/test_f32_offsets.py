"""CPU check of the rule that keeps the float32 kernels' 32-bit row offsets in
range: `f32_offsets_model.cpp` forms the offsets of every lane over window
lengths and positions at the largest row stride that f32_offsets.h lets through
(the header the library takes the rule from)."""

import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2507_02754_amd", "csrc")


def test_offsets_stay_in_range(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path / "f32_offsets_model")
    subprocess.run([gxx, "-std=c++17", "-O1", "-Wall", "-Werror", f"-I{CSRC}",
                    os.path.join(ROOT, "tests", "f32_offsets_model.cpp"), "-o", exe], check=True)
    out = subprocess.run([exe], check=True, capture_output=True, text=True).stdout
    m = re.search(r"violations: (\d+) cases: (\d+) rule: (\w+)", out)
    assert m and int(m.group(1)) == 0 and int(m.group(2)) > 100000 and m.group(3) == "ok", out


def test_library_uses_the_rule():
    src = open(os.path.join(CSRC, "f32.hip")).read()
    assert '#include "f32_offsets.h"' in src
    assert "kFar = static_cast<int>(f32_offsets::kReach)" in src
    api = open(os.path.join(CSRC, "api.hip")).read()
    for call in ("f32_fwd_supported(s)", "f32_bwd_key_supported(s)", "f32_bwd_query_supported(s)"):
        assert call in api, call
