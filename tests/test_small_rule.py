"""Which calls run on the small-block kernel and with how many layers (host rule,
compiled with g++ from paper_2601_16294_amd/csrc/sfc_model.cpp)."""
import itertools
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HARNESS = r'''
#include <stdio.h>
#include <stdlib.h>
#include "sfc_model.h"
int main() {
  long long M, N, K; int ob, ca, ok;
  while (scanf("%lld %lld %lld %d %d %d", &M, &N, &K, &ob, &ca, &ok) == 6) {
    const sfc::SmallChoice s = sfc::small_choose(M, N, K, ob, 256, ca, ok != 0);
    printf("%d %d\n", s.fm, s.layers);
  }
  return 0;
}
'''


@pytest.fixture(scope="module")
def choose(tmp_path_factory):
    d = tmp_path_factory.mktemp("small")
    src, exe = d / "h.cpp", d / "h"
    src.write_text(HARNESS)
    csrc = f"{ROOT}/paper_2601_16294_amd/csrc"
    subprocess.run(["g++", "-std=c++17", "-O1", "-w", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", f"-I{ROOT}/include",
                    f"-I{csrc}", str(src), f"{csrc}/sfc_model.cpp", "-o", str(exe)], check=True)

    def run(calls):
        text = "\n".join(" ".join(str(v) for v in c) for c in calls)
        out = subprocess.run([str(exe)], input=text, capture_output=True, text=True, check=True).stdout.split("\n")
        return [tuple(int(x) for x in line.split()) for line in out if line]
    return run


def test_choices(choose):
    # (M, N, K, output bytes, ca_layers, layers allowed) -> (block rows / 16, layers), 0: curve kernel
    calls = {
        (16, 14336, 4096, 2, 0, 1): (1, 1),
        (1, 4096, 4096, 2, 0, 1): (1, 4),
        (13, 1024, 16384, 2, 0, 1): (1, 8),
        (13, 1024, 16384, 2, 0, 0): (0, 1),      # no memory for layer copies: the curve kernel's
        (13, 1024, 16384, 2, 1, 1): (1, 1),      # one layer asked for
        (32, 14336, 4096, 2, 0, 1): (2, 1),
        (1024, 1024, 1024, 2, 1, 1): (4, 1),
        (128, 128, 65535, 4, 0, 1): (1, 16),
    }
    assert choose(calls.keys()) == list(calls.values())
    for c in [(1024, 2048, 512, 2, 1, 1), (8192, 8192, 8192, 2, 0, 1), (16, 16384, 16384, 2, 0, 1), (64, 64, 7, 4, 1, 1)]:
        assert choose([c])[0][0] == 0, c


def test_one_round(choose):
    # blocks x layers never exceed the CUs, layers only where allowed, and every
    # layer has at least two 64-deep stages per wave
    sides = [1, 16, 17, 33, 64, 100, 256, 1000, 4096, 16384]
    calls = [(M, N, K, 2, ca, ok) for M, N in itertools.product(sides, sides) for K in (8, 500, 4096, 65536)
             for ca, ok in ((0, 1), (0, 0), (1, 1))]
    taken = 0
    for (M, N, K, _, ca, ok), (fm, layers) in zip(calls, choose(calls)):
        if fm == 0:
            continue
        taken += 1
        assert -(-M // (16 * fm)) * -(-N // 64) * layers <= 256
        assert layers == 1 or (ca == 0 and ok == 1 and -(-K // 64) >= 8 * layers)
    assert taken > 100
