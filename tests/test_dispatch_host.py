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


def test_attention_on_few_query_blocks(ask):
    """32-query workgroups fit the chip once, or twice with long rows, whatever its size."""
    shapes = {(1, 1, 64): 2, (16, 4, 4): 2, (13, 1, 5): 1, (2, 1, 47): 1, (2, 1, 48): 2,
              (1, 1, 128): 2, (1, 1, 129): 1, (8, 1, 16): 1}
    got = ask([f"attn {hq} {hkv} {nb} 0 256" for hq, hkv, nb in shapes])
    assert got == list(shapes.values())
    # half the compute units, half the query blocks
    assert ask([f"attn 1 1 {nb} 0 128" for nb in (32, 33, 47, 48, 64, 65)]) == [2, 1, 1, 2, 2, 1]
    for hq, hkv, nb in shapes:  # dense and listed calls alike
        a, b = ask([f"attn {hq} {hkv} {nb} {dense} 256" for dense in (0, 1)])
        assert (a == 2) == (b == 2)


def test_attention_order(ask):
    lists = {(32, 8, 128): 1, (32, 8, 129): 0, (16, 16, 256): 1, (28, 4, 73): 1, (28, 4, 74): 0,
             (64, 8, 32): 1, (10, 2, 205): 0}
    assert ask([f"attn {hq} {hkv} {nb} 0 256" for hq, hkv, nb in lists]) == list(lists.values())
    dense = {(32, 8, 256): 1, (32, 8, 257): 0, (24, 24, 85): 1, (24, 24, 86): 0}
    assert ask([f"attn {hq} {hkv} {nb} 1 256" for hq, hkv, nb in dense]) == list(dense.values())
