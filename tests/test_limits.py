"""The host's rule for emitting a streamed 2D step before the next step's total is known (csrc/limits.h, compiled here):
it holds only where no outcome of that step can push an offset beyond the 32-bit hit indices."""
import os
import random
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIMIT = 2 ** 32 - 2  # hits that the entry points accept

PROGRAM = r"""
#include <cstdio>
#include "limits.h"
int main() {
  long long total, vertices;
  while (std::scanf("%lld %lld", &total, &vertices) == 2) std::printf("%d\n", ftk::step_fits(total, vertices) ? 1 : 0);
}
"""


@pytest.fixture(scope="module")
def step_fits(tmp_path_factory):
    d = tmp_path_factory.mktemp("limits")
    (d / "main.cpp").write_text(PROGRAM)
    inc = os.path.join(ROOT, "paper_2011_08697_amd", "csrc")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-I", inc, "-o", str(d / "main"), str(d / "main.cpp")])

    def ask(pairs):
        text = "".join("%d %d\n" % p for p in pairs)
        out = subprocess.run([str(d / "main")], input=text, capture_output=True, text=True, check=True).stdout.split()
        assert len(out) == len(pairs)
        return [v == "1" for v in out]

    return ask


def test_early_emission_never_sees_an_offset_beyond_the_indices(step_fits):
    rng = random.Random(1)
    pairs = [(0, 4), (0, LIMIT // 12), (0, LIMIT // 12 + 1), (LIMIT, 4), (LIMIT - 48, 4), (LIMIT - 47, 4), (LIMIT, 0),
             (0, 1 << 40), (LIMIT, 1 << 40), (LIMIT - 12 * 4096 ** 2, 4096 ** 2), (LIMIT - 12 * 4096 ** 2 + 1, 4096 ** 2)]
    pairs += [(rng.randrange(LIMIT + 1), int(2 ** rng.uniform(2, 33))) for _ in range(2000)]
    for (total, vertices), got in zip(pairs, step_fits(pairs)):
        assert got == (total + 12 * vertices <= LIMIT), (total, vertices)
