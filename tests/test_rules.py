"""The rules by which a barycenter plan chooses its sweeps (csrc/wts_rules.h), built
with the host compiler.  Rows per lane of the non-allocating score call: a plan
whose score workspace fitted its scratch with the rows of the earlier rule (4, or
5 where that brings more than 13/16 of the SIMDs' strips under it) still fits."""
import os
import shutil
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "..", "paper_2404_12134_amd", "csrc")
SCRATCH = 32 << 20
CUS = 256


@pytest.fixture(scope="module")
def rules_bin(tmp_path_factory):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    exe = str(tmp_path_factory.mktemp("rules") / "rules")
    subprocess.run([cxx, "-std=c++17", "-O1", "-I", CSRC, os.path.join(HERE, "rules_main.cpp"),
                    "-o", exe], check=True)
    return exe


def plans(exe, cases):
    """[(d, L, fp32, team, lengths)] -> [(rho, {rho: workspace bytes})]"""
    return [(r[0], dict(zip((2, 4, 5), r[1:4]))) for r in rules(exe, cases)]


def rules(exe, cases):
    """The rows that rules_main.cpp prints."""
    inp = "\n".join("%d %d %d %d %d %d %s" % (d, L, fp32, team, CUS, len(lens),
                                             " ".join(map(str, lens)))
                    for d, L, fp32, team, lens in cases)
    out = subprocess.run([exe], input=inp, capture_output=True, text=True, check=True).stdout
    return [tuple(map(int, ln.split())) for ln in out.splitlines()]


def earlier_rho(L, n):
    simds = 4 * CUS
    i4, i5, cap = n * -(-L // 256), n * -(-L // 320), simds * 13 // 16
    return 5 if cap < i4 <= 2 * simds and i5 <= cap else 4


def test_plans_at_the_border_of_the_scratch(rules_bin):
    got = plans(rules_bin, [(3, 17560, 0, 1, [3000] * 14), (3, 3072, 0, 1, [3000] * 83)])
    for rho, size in got:
        assert size[5] <= SCRATCH < size[4] and rho == 5


@pytest.mark.parametrize("fp32", [0, 1])
@pytest.mark.parametrize("team", [0, 1])
def test_no_plan_that_fitted_the_scratch_is_refused(rules_bin, team, fp32):
    rng = np.random.default_rng(2 * team + fp32)
    cases = []
    for _ in range(6000):
        n = int(np.exp(rng.uniform(0, np.log(600))))
        L = int(np.exp(rng.uniform(0, np.log(50000))))
        N = int(np.exp(rng.uniform(0, np.log(50000))))
        lens = [N] * n if rng.random() < 0.5 else rng.integers(max(1, N // 2), 2 * N, n).tolist()
        cases.append((int(rng.integers(1, 9)), L, fp32, team, lens))
    lost = fitted = 0
    for (d, L, _, _, lens), (rho, size) in zip(cases, plans(rules_bin, cases)):
        if size[earlier_rho(L, len(lens))] <= SCRATCH:
            fitted += 1
            lost += size[rho] > SCRATCH
    assert fitted > 1000 and lost == 0


def test_waves_and_path_recovery_of_measured_batches(rules_bin):
    """Batches where one choice was measured at least a tenth faster than the
    other; n lengths even between 0.8 N and 1.2 N."""
    values, scores, sub, paths, pairs = range(4, 9)

    def lens(n, N):
        return np.random.default_rng(0).integers(int(0.8 * N), int(1.2 * N) + 1, n).tolist()

    got = rules(rules_bin, [
        (3, 4000, 0, 0, lens(128, 4000)),   # float64 scores: one wave, 1.52 ms against 1.74
        (3, 4000, 1, 0, lens(128, 4000)),   # float32: two, 1.18 against 1.41
        (1, 4000, 0, 0, lens(256, 4000)),   # light Sub-DTW: three, 2.20 against 2.68
        (6, 8000, 0, 0, lens(64, 8000)),    # six channels: one, 3.97 against 5.10
        (1, 1000, 0, 0, lens(2000, 1000)),  # many strips
        (1, 4000, 0, 0, lens(256, 4000)),   # paths from checkpoints, 1.57 against 2.42
        (6, 1000, 0, 0, lens(2000, 1000)),  # from codes, 1.95 against 2.50
    ])
    assert got[0][scores] == 1 and got[1][scores] >= 2 and got[2][sub] == 3 and got[3][scores] == 1
    assert min(got[4][values:pairs]) >= 2
    assert got[5][pairs] == 1 and got[6][pairs] == 0


def test_waves_of_equal_lengths(rules_bin):
    """Strips of equal lengths end together: a second wave on a SIMD of three
    strips was measured to cost there, us at one / two waves."""
    scores, sub = 5, 6
    got = rules(rules_bin, [
        (3, 4000, 0, 0, [4000] * 128),   # float64 scores 1390 / 1674
        (6, 4000, 0, 0, [4000] * 128),   # Sub-DTW 2043 / 2430
        (6, 8000, 0, 0, [8000] * 64),    # 4034 / 5069
        (3, 4000, 1, 0, [4000] * 128),   # float32: two
    ])
    assert got[0][scores] == 1 and got[1][sub] == 1 and got[2][sub] == 1 and got[3][scores] >= 2
