"""The rules by which launches are cut and kernels chosen (launch_rules.h),
built on their own with AddressSanitizer and UndefinedBehaviorSanitizer.  CPU
only."""
import os
import shutil
import subprocess

import numpy as np
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


def test_noise_of_the_weights(rules):
    """The mean error P^-1/2 of the measured links, at most 1 each."""
    rng = np.random.default_rng(5)
    for n in (0, 1, 2, 65, 4097):
        P = np.exp(rng.uniform(-5, 15, n)) * (rng.random(n) < 0.7)
        want = np.minimum(1.0, P[P > 0] ** -0.5).mean() if (P > 0).any() else 0.0
        got = rules(f"noise {n} " + " ".join(float(p).hex() for p in P))[0][0]
        assert abs(got - want) <= 1e-12 * max(1.0, want), n


# chain counts that four lanes per chain take as fast or faster: (model, L,
# staged table, noise of the weights, chains)
FEW = [(0, 64, 1, 0.02, 12288), (0, 64, 1, 0.09, 4160), (0, 64, 1, 0.09, 8192), (0, 48, 1, 0.02, 8256),
       (0, 48, 1, 0.02, 10240), (0, 32, 1, 0.02, 8256), (0, 32, 1, 0.02, 9216), (0, 32, 1, 0.09, 4160),
       (0, 24, 1, 0.02, 8256), (0, 24, 1, 0.02, 8704), (0, 24, 1, 0.1, 8192), (0, 16, 1, 0.02, 8256),
       (0, 16, 1, 0.1, 4160), (0, 8, 1, 0.1, 8192), (0, 64, 0, 0.09, 10240), (0, 64, 0, 0.02, 16384),
       (0, 64, 1, 0.06, 8192), (0, 24, 1, 0.06, 8192), (1, 32, 1, 0.02, 9728),
       (1, 32, 1, 0.19, 4160), (1, 48, 1, 0.19, 8256), (1, 24, 1, 0.2, 6144), (1, 16, 1, 0.19, 8192),
       (1, 8, 1, 0.02, 8256), (1, 8, 1, 0.19, 6144), (1, 4, 1, 0.3, 2048), (1, 4, 1, 0.01, 4096),
       (1, 64, 0, 0.16, 16384), (2, 24, 1, 0.02, 16896), (2, 16, 1, 0.02, 16384)]
# and that one wavefront per chain takes faster
WAVE = [(0, 64, 1, 0.04, 8192), (0, 64, 1, 0.0, 8192), (0, 64, 1, 0.09, 4096), (0, 32, 1, 0.04, 8192),
        (0, 32, 1, 0.1, 4096), (0, 32, 1, 0.06, 8192), (0, 64, 1, 0.06, 6144), (1, 64, 1, 0.2, 12288),
        (0, 8, 1, 0.01, 8192), (1, 48, 1, 0.07, 12288), (1, 48, 1, 0.2, 8192),
        (1, 64, 0, 0.04, 24576), (1, 64, 0, 0.2, 12288), (1, 16, 1, 0.05, 8192), (1, 4, 1, 0.4, 1024),
        (2, 64, 0, 0.3, 40960), (2, 32, 1, 0.3, 20480), (2, 16, 1, 0.03, 14336), (2, 8, 1, 0.05, 12288)]


def test_default_lines(rules):
    got = rules(*(f"line {m} {L} {s} {noise}" for m, L, s, noise, _ in FEW + WAVE))
    for (m, L, s, noise, chains), (_, line) in zip(FEW + WAVE, got):
        assert (chains <= line) == ((m, L, s, noise, chains) in WAVE), (m, L, s, noise, chains, line)


def test_no_line_below_the_chains_that_take_16_lanes(rules):
    """Lattices whose lanes per chain are 16 by default up to 4096 chains
    have one wavefront per chain there, whatever the weights; only Potts
    lattices of L not a multiple of 16 (4 lanes) may lie lower."""
    cases = [(m, L, s, noise) for m in (0, 1, 2) for L in (4, 8, 16, 24, 32, 48, 64) for s in (0, 1)
             for noise in (0.0, 0.06, 1.0)]
    lines = {c: v[1] for c, v in zip(cases, rules(*("line %d %d %d %g" % c for c in cases)))}
    for (m, L, s, noise), line in lines.items():
        if m != 1 or L % 16 == 0:
            assert line >= 4096, (m, L, s, noise)
        assert line <= lines[(m, L, s, 0.0)]


def test_autotuner_times_every_default_workgroup(rules):
    """The workgroups that a run takes by default are among the autotuner's
    candidates, and no launch is timed twice."""
    flat = [int(v) for v in rules("shapes")[0]]
    shapes = list(zip(flat[::2], flat[1::2]))
    launches = [(l, t) if l < 16 else (l, min(16, t // l)) for l, t in shapes]
    assert len(set(launches)) == len(launches), launches
    chains = [1, 64, 1024, 1025, 1536, 2048, 2049, 4096, 20480]
    for n, (tile,) in zip(chains, rules(*(f"tile 16 {n} 256" for n in chains))):
        assert tile == (4 if n <= 1024 else 8 if n <= 2048 else 16), n
        assert (16, 16 * tile) in shapes, n
    assert {(l, 256) for l in (1, 2, 4)} <= set(shapes)
    assert [v for v, in rules("tile 4 4096 256", "tile 64 4096 256")] == [4, 16]


def test_probe_weights(rules):
    """Independent and uniform in (-0.15, 0.15), the same on every call."""
    a, b = np.array(rules("probe 8193", "probe 8193"))
    assert np.array_equal(a, b) and np.all(np.abs(a) < 0.15)
    assert abs(a.mean()) < 5 * 0.15 / np.sqrt(3 * len(a)) and abs(a.std() - 0.15 / np.sqrt(3)) < 0.003
    assert abs(np.corrcoef(a[:-1], a[1:])[0, 1]) < 0.06
