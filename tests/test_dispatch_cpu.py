"""What the library asks of the HIP runtime (allocations, launches), on a runtime that only records: tests/fakehip/.  Each
scenario runs in a process of its own, so that the recorded runtime is the one its library finds."""
import os
import shutil
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
FAKE = os.path.join(ROOT, "tests", "fakehip")


@pytest.fixture(scope="module")
def fake(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("g++ not installed")
    so = str(tmp_path_factory.mktemp("fakehip") / "libfakehip.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-o", so, os.path.join(FAKE, "fake_hip.cpp")], check=True)
    return so


@pytest.mark.parametrize("scenario", ["graph_block_stays", "short_of_memory", "most_tokens", "widest_routed", "smallest_routed",
                                      "unsplit_narrow", "in_place", "decode_gate_up", "decode_down", "decode_few_tokens",
                                      "decode_odd_boundaries", "routed_grid", "float_blocks", "float_token_tiles",
                                      "partial_sums_at_the_limit"])
def test_scenario(fake, scenario):
    from paper_2511_21089_amd import binding as mm
    res = subprocess.run([sys.executable, os.path.join(FAKE, "scenarios.py"), scenario, fake, mm.lib._name],
                         stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=120)
    assert res.returncode == 0 and res.stdout.strip().endswith("ok"), res.stdout[-4000:]
