"""Which calls run on the small-block kernel and with how many layers (host rule,
compiled with g++ from paper_2601_16294_amd/csrc/sfc_model.cpp)."""
import itertools

import pytest

import host_rule


@pytest.fixture(scope="module")
def choose(tmp_path_factory):
    return host_rule.build(str(tmp_path_factory.mktemp("small")), r'''
  long long M, N, K; int ob, ca;
  while (scanf("%lld %lld %lld %d %d", &M, &N, &K, &ob, &ca) == 5) {
    const sfc::SmallChoice s = sfc::small_choose(M, N, K, ob, 256, ca);
    printf("%d %d\n", s.fm, s.layers);
  }''')


def test_choices(choose):
    # (M, N, K, output bytes, ca_layers) -> (block rows / 16, layers), 0: curve kernel
    calls = {
        (16, 14336, 4096, 2, 0): (1, 1),
        (1, 4096, 4096, 2, 0): (1, 4),
        (13, 1024, 16384, 2, 0): (1, 8),
        (13, 1024, 16384, 2, 1): (1, 1),      # one layer asked for
        (32, 14336, 4096, 2, 0): (2, 1),
        (1024, 1024, 1024, 2, 1): (4, 1),
        (128, 128, 65535, 4, 0): (1, 16),
        # large weights: many rounds of K, or rows of B that meet on few channels, leave
        # them to the curve kernel; timed on both sides
        (16, 12520, 7656, 2, 0): (0, 1),
        (1, 12520, 7656, 2, 0): (0, 1),
        (16, 16384, 8192, 2, 0): (0, 1),
        (4, 16384, 6144, 2, 0): (0, 1),
        (16, 12288, 12288, 2, 0): (0, 1),
        (12, 11840, 12352, 2, 0): (1, 1),
        (16, 13376, 6840, 2, 0): (1, 1),
        (16, 13640, 6808, 2, 0): (0, 1),
        (58, 13056, 7680, 2, 0): (0, 1),
        (16, 12288, 8192, 2, 0): (1, 1),
        (33, 16384, 6144, 2, 0): (4, 1),
        (1, 16336, 4712, 2, 0): (1, 1),
        (16, 8192, 8192, 2, 0): (1, 2),
        (3, 3096, 12560, 2, 0): (1, 4),
        (20, 6688, 9280, 2, 0): (2, 2),
        (209, 1464, 9296, 4, 0): (0, 1),
    }
    got = [(fm, layers if fm else 1) for fm, layers in choose(calls.keys())]
    assert got == list(calls.values())
    for c in [(1024, 2048, 512, 2, 1), (8192, 8192, 8192, 2, 0), (16, 16384, 16384, 2, 0), (64, 64, 7, 4, 1)]:
        assert choose([c])[0][0] == 0, c


def test_one_round(choose):
    # blocks x layers never exceed the CUs, layers only where allowed, and every
    # layer has at least two 64-deep stages per wave
    sides = [1, 16, 17, 33, 64, 100, 256, 1000, 4096, 16384]
    calls = [(M, N, K, 2, ca) for M, N in itertools.product(sides, sides) for K in (8, 500, 4096, 65536)
             for ca in (0, 1)]
    taken = 0
    for (M, N, K, _, ca), (fm, layers) in zip(calls, choose(calls)):
        if fm == 0:
            continue
        taken += 1
        assert -(-M // (16 * fm)) * -(-N // 64) * layers <= 256
        assert layers == 1 or (ca == 0 and -(-K // 64) >= 8 * layers)
    assert taken > 100
