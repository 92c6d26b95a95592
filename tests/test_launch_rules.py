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
