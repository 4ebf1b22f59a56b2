"""The key searches of the COPASS partition, on the host: each ends at the
smallest key at or past the one it seeks and never leaves the range it began
with, also when the other search still goes on and when no key of the range
is the sought one."""
import os
import random
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2306_09855_amd", "csrc")


@pytest.fixture(scope="module")
def probe(tmp_path_factory):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    exe = str(tmp_path_factory.mktemp("probe") / "probe")
    subprocess.run([hipcc, "-O1", "-I", CSRC, "-o", exe, os.path.join(HERE, "partition_search_probe.cpp")],
                   check=True, capture_output=True)
    return exe


def test_searches_end_inside_their_range(probe):
    rng = random.Random(3)
    top = 2 ** 32 - 1
    cases = []
    for k in range(4000):
        width = int(2 ** rng.uniform(0, 32)) if k % 3 else rng.choice([9, 81, 729, 6561, 59049]) + rng.randrange(2)
        a = rng.choice([0, rng.randrange(max(1, top - width)), max(0, top - width)])
        b = min(top, a + width)
        # the upper bounds reach m at b or before; the lower ones later, perhaps nowhere
        f0 = rng.choice([a, b, rng.randint(a, b)])
        f1 = rng.choice([top + 1, top + 1, b, rng.randint(f0, b)])
        cases.append((a, b, f0, f1))
    out = subprocess.run([probe], input="\n".join(" ".join(map(str, c)) for c in cases), check=True,
                         capture_output=True, text=True).stdout.split("\n")
    for (a, b, f0, f1), line in zip(cases, out):
        a0, b0, a1, b1, rounds = map(int, line.split())
        assert (a0, b0) == (f0, f0), (a, b, f0, f1)
        assert (a1, b1) == (min(f1, b),) * 2, (a, b, f0, f1)
        assert rounds <= 11
