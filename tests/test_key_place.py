"""Where the survivors' sort places a key (key_top32, key_place of kc_segsort.hpp), compiled for the
host: the leading 32 of a key's bits for keys of every width, wide keys of a few bits among them
(set << 2k | k-mer: 2k + 1 bits and more in two words), under UndefinedBehaviorSanitizer."""
import os
import random
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


def test_places(tmp_path):
    if shutil.which(HIPCC) is None:
        pytest.skip("no hipcc")
    exe = str(tmp_path / "key_place")
    subprocess.run([HIPCC, "-x", "hip", "--offload-arch=gfx950", "-O1", "-std=c++17", "-Xclang",
                    "-target-feature", "-Xclang", "-packed-fp32-ops", "-Xarch_host", "-fsanitize=undefined",
                    "-Xarch_host", "-fno-sanitize-recover=all", "-o", exe, os.path.join(HERE, "key_place.cpp")],
                   check=True, capture_output=True)
    rng = random.Random(5)
    keys = []
    for words, top in ((1, 62), (2, 126)):
        for nbits in range(2, top + 1):
            for x in {0, 1, (1 << nbits) - 1, 1 << (nbits - 1)} | {rng.getrandbits(nbits) for _ in range(20)}:
                keys.append((words, nbits, x))
    text = "".join(f"{w} {n} {x >> 64:x} {x & ((1 << 64) - 1):x}\n" for w, n, x in keys)
    run = subprocess.run([exe], input=text, capture_output=True, text=True)
    assert run.returncode == 0, run.stderr[-2000:]
    lines = run.stdout.splitlines()
    assert len(lines) == len(keys)
    for (w, n, x), line in zip(keys, lines):
        t = x >> (n - 32) if n >= 32 else x << (32 - n)
        c = 0xFFFFFFFF - ((0xFFFFFFFF - t) ** 2 >> 32)
        assert [int(v) for v in line.split()] == [t, t, c], f"{w} words, {n} bits, key {x:x}"
