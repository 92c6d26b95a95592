"""How launches are split (csrc/launch_rules.h), evaluated on the CPU: the
rules are built with g++ together with a small driver
(tests/sanitize/launch_rules_driver.cpp) and queried."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2605_07612_amd", "csrc")


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path_factory.mktemp("rules") / "driver")
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-fsanitize=address,undefined", "-I" + CSRC,
                        os.path.join(ROOT, "tests", "sanitize", "launch_rules_driver.cpp"), "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]

    def run(*queries):
        text = "\n".join(" ".join(str(x) for x in q) for q in queries) + "\n"
        r = subprocess.run([exe], input=text, capture_output=True, text=True,
                           env=dict(os.environ, ASAN_OPTIONS="detect_leaks=0"))
        assert r.returncode == 0, r.stderr[-2000:]
        return [int(x) for x in r.stdout.split()]
    return run


def test_configured_slabs_are_what_runs(ask):
    """k-slabs that a caller configures are taken as they are (of 8 planes or
    more), however few blocks there are; with none configured, the model's."""
    q = [(c, N, p) for c in (1, 2, 4) for N in (8, 16, 32) for p in (1, 2, 4, 8, 16, 32)]
    assert ask(*[("slabs", *x) for x in q]) == [min(c, N // 8) for c, N, _ in q]
    q = [(0, N, p) for N in (8, 16, 32) for p in (1, 2, 4, 8, 16, 32)]
    assert ask(*[("slabs", *x) for x in q]) == [max(1, N // p) for _, N, p in q]


def test_model_planes(ask):
    """The depth that the model takes on a device of 256 CUs for the block
    counts that were swept."""
    swept = [(0, 16, 180, 4), (0, 16, 512, 8), (0, 16, 720, 16), (0, 32, 80, 16), (0, 32, 1, 1), (1, 16, 180, 8),
             (1, 32, 27, 8), (0, 8, 512, 2), (0, 16, 4096, 16), (1, 16, 4096, 16), (0, 32, 512, 32)]
    assert ask(*[("planes", f64, 256, 1, N, nb) for f64, N, nb, _ in swept]) == [x[3] for x in swept]
    assert ask(("planes", 0, 256, 3, 8, 19270, 16, 6937, 32, 12333)) == [32]


def test_rules_follow_the_compute_units(ask):
    """Every rule fills the device it runs on: the block counts that were swept
    on 256 CUs take the measured split there, and a device of a fourth of the
    CUs splits a fourth of the blocks or records alike, so that it does not pay
    for slabs that it cannot run at once."""
    swept = [("weno", 80, 32, 8), ("weno", 512, 16, 8), ("weno", 512, 8, 4), ("weno", 4, 32, 1),
             ("advect", 180, 16, 2), ("advect", 512, 8, 0), ("advect", 80, 32, 1), ("advect", 28, 32, 3),
             ("ghost", 448, 5 * 2 * 256, 4), ("ghost", 4096, 5 * 2 * 256, 1), ("ghost", 4, 5 * 2 * 256, 5)]
    assert ask(*[(w, n, x, 256) for w, n, x, _ in swept]) == [e for _, _, _, e in swept]
    assert ask(*[(w, n // 4, x, 64) for w, n, x, _ in swept]) == [e for _, _, _, e in swept]
    many = [("planes", p, cu, 1, N, cu // 64 * nb) for p in (0, 1) for N in (8, 16, 32) for nb in (3, 45, 128, 700)
            for cu in (256, 64)]
    got = ask(*many)
    assert got[::2] == got[1::2]
