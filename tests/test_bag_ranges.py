"""Bag offsets that hold anything at all must not lead a kernel outside its buffers: the range arithmetic
of the kernels, compiled for the host, against the same rules in Python's integers."""
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def check(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("bags") / "bag_ranges_check")
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    subprocess.check_call([hipcc, "-x", "hip", "--offload-host-only", "--offload-arch=gfx950", "-O1", "-std=c++17",
                           os.path.join(ROOT, "tests", "bag_ranges_check.cpp"), "-o", exe])

    def run(cases):
        text = "\n".join("%d %d %s" % (n, len(off) - 1, " ".join(str(int(x)) for x in off)) for n, off in cases)
        out = subprocess.run([exe], input=text, capture_output=True, text=True, timeout=60, check=True).stdout
        return [line.split() for line in out.splitlines()]
    return run


def _violations(n, off):
    return sum(1 for b in range(len(off) - 1)
               if off[b + 1] < off[b] or (b == 0 and off[0] != 0) or (b == len(off) - 2 and off[-1] != n))


def test_ranges_stay_inside_whatever_the_offsets_hold(check):
    n, nb = 1000, 200
    good = np.linspace(0, n, nb + 1).astype(np.int64).tolist()
    big = [2 ** 63 - 1, -2 ** 63, 2 ** 31, 2 ** 32 + 500, -2 ** 31 - 1, -2 ** 32 + 100, -0x180000001, -7, n + 1]
    cases = [(n, good), (n, [0] + [n] * nb), (n, [0] * nb + [n]), (0, [0] * (nb + 1)), (1, [0, 1]), (7, [0, 7])]
    for x in big:
        cases += [(n, [0] + [x] * (nb - 1) + [n]),               # every inner offset: inner wavefronts see no violation
                  (n, [x] * (nb + 1)), (n, [x] + good[1:]), (n, good[:-1] + [x]),
                  (n, good[:70] + [x] * 60 + good[130:]),        # a whole wavefront's bags
                  (n, good[:100] + [x] + good[101:]), (n, good[:128] + [x] + good[129:])]
    rng = np.random.default_rng(1)
    for _ in range(200):                                          # runs of good offsets and of anything
        off = list(good)
        for _ in range(rng.integers(1, 5)):
            a, m = int(rng.integers(0, nb + 1)), int(rng.integers(1, 90))
            v = sorted(int(rng.choice(big)) + int(rng.integers(0, 50)) if rng.random() < 0.3 else int(rng.integers(-n, 2 * n))
                       for _ in range(min(m, nb + 1 - a)))
            off[a:a + len(v)] = [max(-2 ** 63, min(2 ** 63 - 1, x)) for x in v]
        cases.append((n, off))
    for (m, off), (bad, verdict) in zip(cases, check(cases)):
        assert verdict == "ok" and int(bad) == _violations(m, off), (m, off, bad, verdict)
