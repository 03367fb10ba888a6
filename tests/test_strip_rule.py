"""When 256x256 blocks with a half-height strip take over from the model's 128x256
blocks (host rule, compiled with g++ from paper_2601_16294_amd/csrc/sfc_model.cpp)."""
import itertools

import pytest

import host_rule


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    return host_rule.build(str(tmp_path_factory.mktemp("strip")), r'''
  long long M, N, K; int ob;
  const int occ[4] = {2, 1, 1, 1};
  while (scanf("%lld %lld %lld %d", &M, &N, &K, &ob) == 4) {
    const sfc::ModelChoice ch = sfc::model_choose(M, N, K, ob, 256, occ, -1, 1);
    const long long gm = (M + 255) / 256, gn = (N + 255) / 256;
    printf("%d %d %d\n", ch.tile == sfc::kT128x256, (int)sfc::strip_beats_128x256(M, N, (K + 63) / 64, ob, 256, ch),
           sfc::strip_columns((int)gm, (int)gn, 256, (M + 127) / 128, 256));
  }''')


def test_measured_shapes(rule):
    yes = [(6144, 6144, 4096, 2), (6144, 6144, 4096, 4), (5120, 4096, 8192, 2), (1300, 14336, 4096, 2),
           (3001, 7003, 5001, 2), (2560, 14336, 4096, 2), (5500, 4096, 4096, 2), (4096, 6144, 4096, 4)]
    no = [(3000, 7000, 2048, 4), (3000, 7000, 2048, 2), (2800, 6144, 4096, 2), (3300, 6144, 4096, 2),
          (8192, 8192, 8192, 2), (4096, 14336, 4096, 2), (1024, 2048, 512, 2)]
    assert all(r[1] == 1 for r in rule(yes))
    assert all(r[1] == 0 for r in rule(no))


def test_only_with_a_strip(rule):
    # never without a strip to launch, nor over another shape than 128x256
    sides = list(range(500, 9000, 613))
    calls = [(M, N, K, 2) for M, N in itertools.product(sides, sides) for K in (600, 4096, 9000)]
    res = rule(calls)
    assert all(t == 1 and w > 0 for t, take, w in res if take)
    assert sum(take for _, take, _ in res) > 10
