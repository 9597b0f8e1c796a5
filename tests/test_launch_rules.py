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
    """The mean error P^-1/2 of the measured links, at most 1 each, over at
    most 1024 evenly spaced ones."""
    rng = np.random.default_rng(5)
    for n in (0, 1, 2, 65, 1024, 1025, 4097, 8193):
        P = np.exp(rng.uniform(-5, 15, n)) * (rng.random(n) < 0.7)
        Q = P[::max(1, -(-n // 1024))]
        want = np.minimum(1.0, Q[Q > 0] ** -0.5).mean() if (Q > 0).any() else 0.0
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
        assert lines[(m, L, s, 1.0)] <= line <= lines[(m, L, s, 0.0)]


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


def round_line(runs, may4=1, may16=1, max_items=4096, cus=256, side=1.0):
    return f"round {may4} {may16} {max_items} {cus} {side} {len(runs)} " + " ".join("%d %r %r" % r for r in runs)


def length(items, cus, side):
    """Length of a round of (number of items, time of each)."""
    n = sum(k for k, _ in items)
    out = max([max(t for _, t in items), sum(k * t for k, t in items) / (cus * side)])
    return max(out, -(-n // cus) * min(t for _, t in items) / side) if n > cus else out


SHARE = {16: 1.0, 8: 0.75, 4: 0.55}


def best_tiles(runs, max_items, cus):
    """(estimate, chains per item) over the three item lengths of the longest run."""
    longest = max(t for _, _, t in runs)
    out = []
    for c in (16, 8, 4):
        within = [next(k for k in (16, 8, 4) if k == 4 or t * SHARE[k] <= 1.001 * longest * SHARE[c])
                  for _, _, t in runs]
        items = [(-(-n // k), t * SHARE[k]) for (n, _, t), k in zip(runs, within)]
        if sum(k for k, _ in items) <= max_items:
            out.append((length(items, cus, 1.0), within))
    return out


def test_no_item_is_shorter_for_sharing_its_cu(rules):
    """12288 chains in 192 items of 64: each has a CU of its own, and the
    round takes what one takes, whatever two do side by side."""
    runs = [(12288, 110.0, 34.0)]
    assert rules(round_line(runs, side=1.3))[0][0] == 1          # 3 rounds of 34 against 110
    assert rules(round_line([(12288, 101.0, 34.0)], side=1.3))[0][0] == 0
    assert rules(round_line([(512 * 64, 100.0, 20.0)], side=1.3))[0][0] == 0  # 154 against 160
    assert rules(round_line([(512 * 64, 100.0, 20.0)], side=1.0))[0][0] == 1  # 200 against 160


def test_a_kernel_that_any_run_rejected_is_not_taken(rules):
    ok, no4, no16 = (640, 110.0, 34.0), (640, -1.0, 34.0), (640, 110.0, -1.0)
    got = rules(round_line([ok, no4]), round_line([ok, no16]), round_line([no4, no16]),
                round_line([ok, no4], max_items=70), round_line([ok, ok], max_items=70),
                round_line([ok, ok], max_items=19), round_line([ok, no16], max_items=19),
                round_line([ok], may4=0, max_items=39), round_line([ok], may4=0, max_items=40),
                round_line([ok], may16=0))
    assert [g[0] for g in got] == [1, 0, -2, -1, 0, -1, -1, -1, 1, 0]
    assert got[1][1:] == [64, 110.0, 64, 110.0]


def test_rounds_take_the_shorter_estimate(rules):
    rng = np.random.default_rng(9)
    cases = []
    for _ in range(300):
        n = int(rng.integers(1, 9))
        runs = [(int(np.exp(rng.uniform(0, 10.5))), float(t), float(t * rng.uniform(0.1, 0.6)))
                for t in np.exp(rng.uniform(0, 4, n))]
        cases.append((runs, int(rng.choice([64, 512, 4096, 100000])), float(rng.choice([1.0, 1.3]))))
    for (runs, max_items, side), got in zip(cases, rules(*(round_line(r, max_items=m, side=s) for r, m, s in cases))):
        four = [(-(-n // 64), t) for n, t, _ in runs]
        four = length(four, 256, side) if sum(k for k, _ in four) <= max_items else None
        tiles = best_tiles(runs, max_items, 256) if sum(-(-n // 16) for n, _, _ in runs) <= max_items else []
        if not tiles and four is None:
            assert got[0] == -1
            continue
        best = min((e for e, _ in tiles), default=None)
        if best is None or (four is not None and four < 0.999 * best):
            assert got[0] == 0, (runs, max_items, side)
        elif four is None or four > 1.001 * best:
            assert got[0] == 1, (runs, max_items, side)
        if got[0] == 1:  # an estimate within 0.1 % of the shortest
            within = [int(k) for k in got[1::2]]
            assert any(w == within and e <= 1.002 * best for e, w in tiles)
            assert got[2::2] == pytest.approx([t * SHARE[k] for (_, _, t), k in zip(runs, within)])
        else:
            assert got[1:] == [v for _, t, _ in runs for v in (64, t)]
