"""The rules on bucket numbers (kc_rules.hpp), in plain host code: the autotuner tries the setting
that a count has without it, whatever the minimizers, and its neighbours; the rule for minimizers of 9
bases and more never takes more buckets than the other, whose number the workspace is sized for."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


def test_the_default_is_among_the_tuners_choices(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("no C++ compiler")
    exe = str(tmp_path / "rules")
    subprocess.run(["g++", "-O1", "-std=c++17", "-o", exe, os.path.join(HERE, "bucket_rules.cpp")], check=True)
    asks = [(kw, n + d, m) for kw in (1, 2) for e in range(10, 33) for n in (1 << e, 3 << (e - 1)) for d in (-1, 0, 1)
            for m in (1, 5, 8, 9, 15, 21)]
    out = subprocess.run([exe], input="".join(f"{a} {b} {c}\n" for a, b, c in asks), capture_output=True, text=True,
                         check=True).stdout.splitlines()
    default = {}
    for ask, line in zip(asks, out):
        v = [int(x) for x in line.split()]
        choices = set(zip(v[1::2], v[2::2]))
        assert {(1, max(1, min(20, v[0] + d))) for d in (-1, 0, 1)} <= choices, ask
        default[ask] = v[0]
    for kw, n, m in asks:
        assert default[(kw, n, m)] <= default[(kw, n, 1)]
        assert default[(kw, n, m)] == default[(kw, n, 9 if m >= 9 else 1)]
