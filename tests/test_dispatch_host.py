"""The dispatch rules, on the host: tests/dispatch_check.cpp compiled host-only
against the library's own header."""
import itertools
import os
import subprocess

import pytest

from .score_tiles import CASES, CUS

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    hipcc = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "bin", "hipcc")
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    exe = tmp_path_factory.mktemp("dispatch") / "dispatch_check"
    cmd = [hipcc, "-x", "hip", "--cuda-host-only", "-O1", "-std=c++17",
           "-I", os.path.join(ROOT, "include"),
           "-I", os.path.join(ROOT, "paper_2503_16428_amd", "csrc"),
           os.path.join(ROOT, "tests", "dispatch_check.cpp"), "-o", str(exe)]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr

    def run(lines):
        out = subprocess.run([str(exe)], input="\n".join(lines), capture_output=True, text=True,
                             timeout=60, check=True).stdout.split()
        assert len(out) == len(lines)
        return [int(x) for x in out]
    return run


def test_the_scoring_cases_cover_every_kernel(ask):
    got = ask([f"score {S} {int(c)} {hq} {nb} {CUS}" for S, c, _, hq, nb in CASES])
    assert got == [tile for _, _, tile, _, _ in CASES]
    assert {c[:3] for c in CASES} == set(itertools.product((1, 2, 4, 8, 16, 32, 64), (True, False),
                                                           (256, 128, 64, 32)))
    for S, _, tile, _, nb in CASES:
        rows = nb * 128 // S
        assert rows > tile and (rows % tile or 128 // S % tile == 0)
