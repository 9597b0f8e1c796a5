"""The rules by which launches are cut and kernels chosen (launch_rules.h),
built on their own with AddressSanitizer and UndefinedBehaviorSanitizer.  CPU
only."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1312_2213_amd", "csrc")


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    d = tmp_path_factory.mktemp("launch_rules")
    subprocess.check_call([gxx, "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
                           "-I", os.path.join(ROOT, "include"), os.path.join(CSRC, "launch_rules_check.cpp"),
                           "-o", str(d / "check")])

    def run(*lines):
        (d / "cases.txt").write_text("\n".join(lines) + "\n")
        r = subprocess.run([str(d / "check"), str(d / "cases.txt")], capture_output=True, text=True, timeout=120)
        assert r.returncode == 0, r.stdout[-500:] + r.stderr
        return [[float(t) for t in line.split()] for line in r.stdout.splitlines()]
    return run


@pytest.mark.parametrize("at_most", [1023, 4095, 65535])
@pytest.mark.parametrize("total", [0, 1, 4094, 4095, 4096, 131071, 2**31 - 1 - 65535, 2**31 - 2, 2**31 - 1])
def test_segments_cover_every_sweep_count(rules, total, at_most):
    """Segments follow each other, end, and add up: up to the longest launch
    that a batched round accepts (2^31 - 1 sweeps), whose end plus one segment
    lies beyond 32 bits."""
    k, total_of, shortest, longest, before = rules(f"segments {total} {at_most}")[0]
    assert (k, total_of) == (-(-total // at_most), total)
    assert longest == min(total, at_most)
    assert shortest == (((total - 1) % at_most + 1) if total else 0)
    assert before == (total - shortest if total else 0)
