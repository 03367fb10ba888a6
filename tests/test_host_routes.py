"""Which kernels, memory and layer counts a call takes: the host layer run against a
stand-in for the HIP runtime (tests/host_api.py), so no GPU is needed."""
import pytest

import host_api
from host_api import gemm

LOAD_ELEMENTS = 0


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    return host_api.build(str(tmp_path_factory.mktemp("host_api")))


def launches(events, *names):
    return [(n, e) for n, e in events if n in (names or ("gemm", "small", "reduce"))]


# fp8 calls with K = 0 are accepted with any N, and the fp8 kernels store 4 columns or
# 16 bytes at a time, which N a multiple of 16 keeps inside C: they may not see
# another N
@pytest.mark.parametrize("M,N,ldc", [(3, 5, 5), (3, 20, 24), (300, 257, 264), (70, 96, 96)])
@pytest.mark.parametrize("tile", [0, 3, 4])
def test_fp8_kernels_only_see_whole_chunks(exe, M, N, ldc, tile):
    calls = host_api.run(exe, [gemm("f8", M, N, 0, out, ca, tile, lda=0, ldb=N, ldc=ldc) for out in (0, 1) for ca in (0, 1, 3)])
    for events in calls:
        assert events[-1] == ("ret", {"rc": 0})
        g = launches(events)
        assert len(g) == 1 and g[0][0] == "gemm"
        assert g[0][1]["f8"] == 0 or N % 16 == 0, g
        assert (g[0][1]["M"], g[0][1]["N"], g[0][1]["K"]) == (M, N, 0)
