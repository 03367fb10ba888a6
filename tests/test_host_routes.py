"""Which kernels, memory and layer counts a call takes: the host layer run against a
stand-in for the HIP runtime (tests/host_api.py), so no GPU is needed."""
import pytest

import host_api
from host_api import gemm


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


# calls that sum layer copies in library memory, and larger ones of the same kind:
# the small-block kernel, the separate reduction, the fused one
LAYERED = {
    "small": (gemm("ex", 13, 1024, 16384, ca=0), gemm("ex", 128, 128, 65535, ca=0), "small"),
    "separate": (gemm("ex", 600, 700, 4096, ca=4), gemm("ex", 1600, 1700, 4096, ca=4), "gemm"),
    "fused": (gemm("fused", 600, 700, 4096, ca=4), gemm("fused", 16000, 17000, 4096, ca=4, tile=1), "gemm"),
    "model": (gemm("ex", 512, 512, 32768, ca=0), gemm("ex", 1024, 1024, 65536, ca=0), "gemm"),
}


def memory(events, kernel):
    e = launches(events, kernel)[0][1]
    return {e["W"] if kernel == "small" else e["out"]} | ({e["counters"]} if e["counters"] else set())


# a recorded call takes the layers of the call that runs at once, whether the stream
# has library memory or not, and memory of its own that nothing frees, whatever grows
@pytest.mark.parametrize("kind", LAYERED)
@pytest.mark.parametrize("warm", [False, True])
def test_captured_calls_own_their_memory(exe, kind, warm):
    small, large, kernel = LAYERED[kind]
    other = [c[:-1] + "2" for c in (small, large)]                    # curve tables, from another stream
    lines = other + ([small] if warm else []) + ["capture 1 1", small, "capture 1 0", small, large, "capture 1 1", large,
                                                 "capture 1 0", large, small]
    calls = host_api.run(exe, lines)
    assert all(c[-1] == ("ret", {"rc": 0}) for c in calls)
    at = len(other) + (1 if warm else 0)
    cap1, eager1, eager2, cap2, eager3, eager4 = (calls[at + i] for i in (1, 3, 4, 6, 8, 9))
    for cap, eager in ((cap1, eager1), (cap2, eager2)):
        a, b = launches(cap, kernel)[0][1], launches(eager, kernel)[0][1]
        assert a["layers"] == b["layers"] > 1
        assert not [e for n, e in cap if n in ("malloc_in_graph", "malloc_async", "free")]
        # counters are zero when the launch starts: cleared in the graph itself
        if a["counters"]:
            names = [n for n, _ in cap]
            assert [e["p"] for n, e in cap if n == "fill"] == [a["counters"]]
            assert names.index("fill") < names.index(kernel)
    held = memory(cap1, kernel) | memory(cap2, kernel)
    for e in (eager1, eager2, eager3, eager4):
        assert not memory(e, kernel) & held
    assert not held & {e["p"] for c in calls for n, e in c if n == "free"}
    if kind != "fused":    # (its larger call grows both)
        sizes = [e["n"] for n, e in cap1 + cap2 if n == "malloc" and e["p"] in held and e["p"] != launches(cap1, kernel)[0][1]["counters"]]
        assert len(sizes) == 2 and sizes[1] >= 2 * sizes[0]


# an allocation that fails in a capture is reported, leaves the thread's capture mode
# as it was (the stand-in's `capture` checks it) and the next call works
def test_captured_allocation_failure(exe):
    small = LAYERED["small"][0]
    calls = host_api.run(exe, ["capture 1 1", "fail 1", small, "capture 1 0", "capture 1 1", small, "capture 1 0", small])
    assert [c[-1][1]["rc"] for c in calls] == [0, 0, -4, 0, 0, 0, 0, 0]
    assert not launches(calls[2])


def model_shape(M, N, K, out):
    """The model's block shape (SFC_TILE_*, layers) with one layer, at the kernels' occupancy."""
    from paper_2601_16294_amd import sfcgemm as sg
    return sg.sfc_gemm_model(M, N, K, out="bf16" if out else "f32", ca_layers=1)["tile"]


# 256x256 blocks take over from the model's 128x256 blocks only together with the
# half-height strip (unaligned operands: a strip of fewer than 8 columns is refused)
@pytest.mark.parametrize("M,N,K", [(2468, 13057, 4096), (2468, 13063, 4096), (2468, 13064, 4096), (2468, 13056 + 255, 4096),
                                   (1300, 14337, 4096), (1300, 14345, 4096), (2561, 8001, 4099), (2561, 7937, 4099)])
def test_whole_blocks_only_with_their_strip(exe, M, N, K):
    for out in (0, 1):
        assert model_shape(M, N, K, out) == "128x256"
        g = [e for _, e in launches(host_api.run(exe, [gemm("ex", M, N, K, out)])[0])]
        tiles = [e["tile"] for e in g]
        assert tiles in ([2], [3, 2]), tiles
        assert sum(e["N"] for e in g) == N and all(e["N"] >= 8 for e in g)


# the strip of fp8 calls, by full rounds, remainder and depth: taken where it gains on
# the mean of the cards that timed it, else one launch
@pytest.mark.parametrize("rounds,K,strip", [
    ((3, 8), 4096, True), ((3, 8), 8192, True), ((3, 8), 3072, False), ((3, 8), 512, False),
    ((3, 4), 4096, True), ((3, 4), 2048, True), ((3, 4), 1024, False), ((3, 4), 256, False),
    ((3, 2), 8192, True), ((3, 2), 4096, False), ((3, 1), 2048, False), ((4, 2), 1024, False),
    ((2, 4), 4096, True), ((2, 8), 3072, True), ((3, 12), 4096, False), ((4, 0), 4096, False)])
def test_fp8_strip(exe, rounds, K, strip):
    M, N = 4096, 256 * (16 * rounds[0] + rounds[1])
    for out in (0, 1):
        g = [e for _, e in launches(host_api.run(exe, [gemm("f8", M, N, K, out)])[0])]
        assert [e["tile"] for e in g] == ([3, 2] if strip else [3]), (rounds, K, out)
        assert sum(e["N"] for e in g) == N and all(e["f8"] == 1 for e in g)


# no strip without the 256x256 blocks it belongs to: a short fp8 call keeps the shape of
# the model where the strip would not pay
def test_fp8_shape_without_a_strip(exe):
    for K in (1024, 2048):
        for w in range(1, 17):
            for R in (1, 2):
                M, N = 4096, 256 * (16 * R + w)
                g = [e["tile"] for _, e in launches(host_api.run(exe, [gemm("f8", M, N, K, 1)])[0])]
                assert len(g) == 1


# the loads that the tests of each path mean to reach, and which calls of theirs run on
# the small-block kernel
def test_load_paths(exe):
    def one(*a, **k):
        return launches(host_api.run(exe, [gemm("ex", *a, **k)])[0])[0]
    ELEMENTS, RING, ANY = 0, 1, 2
    for tile in (1, 2, 3, 4):
        assert one(300, 264, 520, tile=tile, lda=528, ldb=272)[1]["loads"] == RING
        assert one(300, 264, 520, tile=tile, lda=531, ldb=277)[1]["loads"] == ANY
        assert one(300, 264, 520, tile=tile, lda=1 << 20)[1]["loads"] == ELEMENTS
        assert one(300, 264, 520, tile=tile, ldb=1 << 22)[1]["loads"] == ELEMENTS
        for c in (1, 3):
            assert one(300, 7, 520, ca=c, tile=tile)[1]["loads"] == ELEMENTS
            assert one(270, 300, 7, ca=c, tile=tile)[1]["loads"] == ELEMENTS
    for entry in ("ex", "fused"):
        for M, N, K, ca, kernel in ((256, 192, 8192, 0, "small"), (256, 192, 8192, 1, "small"), (300, 200, 12288, 0, "small"),
                                    (520, 512, 16384, 0, "gemm"), (520, 1100, 6144, 0, "gemm"), (700, 2000, 4200, 0, "gemm"),
                                    (1100, 1100, 1000, 0, "gemm"), (1100, 1100, 1000, 1, "gemm")):
            name, e = launches(host_api.run(exe, [gemm(entry, M, N, K, ca=ca)])[0])[0]
            assert name == kernel and (ca == 1 or (M, N) == (1100, 1100) or e["layers"] > 1), (M, N, K, ca)
        # a caller's workspace gets the model's copies
        assert launches(host_api.run(exe, [gemm(entry, 256, 192, 8192, ca=0, ws=1)])[0])[0][0] == "gemm"


# a recorded call whose block grid has no finished curve table yet (the first call of a
# grid, or one whose generator may still run) records the generator and writes a table
# that only recorded calls use; a finished table is used as it is
@pytest.mark.parametrize("call", [gemm("ex", 900, 1300, 600, tile=3), gemm("ex", 4000, 14000, 1000), gemm("ex", 16, 12520, 7656, ca=0)])
def test_recorded_calls_without_a_curve_table(exe, call):
    lines = ["capture 1 1", call, call, "capture 1 0", call, "notready 1", "capture 1 1", call, "capture 1 0", "notready 0",
             "capture 1 1", call, call, "capture 1 0", call]
    calls = host_api.run(exe, lines)
    assert all(c[-1] == ("ret", {"rc": 0}) for c in calls)
    cold, again, eager, pending, done, done2, last = (calls[i] for i in (1, 2, 4, 7, 11, 12, 14))

    def tables(events):
        return [e["table"] for n, e in events if n == "gemm"]

    def orders(events):
        return [e["d"] for n, e in events if n == "order"]
    for c in (cold, again, pending):
        assert orders(c) == tables(c) and len(set(tables(c))) == len(tables(c))
        assert tables(c) == tables(cold)
    assert not set(tables(eager)) & set(tables(cold)) and orders(eager) == tables(eager)
    for c in (done, done2, last):
        assert tables(c) == tables(eager) and not orders(c)
    assert not [e for n, e in again + pending + done if n == "malloc"]
