"""The small-block kernel (few rows, small products): block edges, every row-end
remainder, half stages and register steps, layers within and across waves.
Integer operands make every sum exact in fp32 (|sum| <= 16 K < 2^24), so results are
compared bit for bit; padding holds NaN, so an element used from outside a row
shows.  (sizes below are ones the library gives to this kernel, see
test_small_rule.py)"""
import numpy as np
import pytest
import torch

from oracle import bf16 as obf16
from paper_2601_16294_amd.inputs import draw
from gpu_util import run_gemm, to_host, upload, sg

pytestmark = pytest.mark.gpu


def want_of(A, B, K, N, out):
    w = (obf16.bf16_to_f64(A[:, :K]) @ obf16.bf16_to_f64(B[:, :N])).astype(np.float32)   # exact: integers < 2^24
    return obf16.bf16_to_f64(obf16.f32_to_bf16_rne(w)) if out == "bf16" else w.astype(np.float64)


def check(M, N, K, c, out, lda, ldb, ldc, seed):
    A = draw(M, K, ("int", -4, 4), seed, lda)
    B = draw(K, N, ("int", -4, 4), seed + 1, ldb)
    C = run_gemm(A, B, M, N, K, out=out, ldc=ldc, ca_layers=c, tile="auto")
    assert np.array_equal(C[:, :N], want_of(A, B, K, N, out)), (M, N, K, c, out)
    assert np.isnan(C[:, N:]).all()


# rows around the 16, 32 and 64-row blocks, aligned and not
@pytest.mark.parametrize("M", [1, 15, 16, 17, 33, 64, 65, 200])
def test_rows(M):
    check(M, 520, 320, 1, "bf16", 320, 520, 520, 3000 + M)
    check(M, 61, 333, 0, "f32", 335, 63, 62, 3100 + M)


# K at the edges of the 32-deep step, the 64-deep stage and the four waves' turns;
# N with every remainder of a chunk and of the 64-column block
@pytest.mark.parametrize("K", [8, 9, 31, 32, 33, 63, 64, 65, 96, 127, 128, 160, 255, 256, 257, 288, 321, 512, 1000])
def test_depths(K):
    check(37, 136, K, 1, "f32", (K + 7) // 8 * 8, 136, 136, 3200 + K)
    check(18, 64 + K % 9, K, 1, "bf16", K, 64 + K % 9, 64 + K % 9, 3300 + K)


@pytest.mark.parametrize("N", list(range(8, 17)) + [63, 64, 65, 127, 129])
def test_columns(N):
    check(20, N, 192, 1, "f32", 192, N, N + 1, 3400 + N)
    check(500, N, 77, 0, "bf16", 77, N + 2, N, 3500 + N)


# layers (the library's choice): the last workgroup of a block sums the copies; the
# counters are zero again, so that calls repeat; block heights of 16, 32 and 64
@pytest.mark.parametrize("M,N,K", [(13, 1024, 16384), (1, 512, 8191), (60, 1000, 16000), (128, 128, 65535),
                                   (256, 256, 8192)])
def test_layers(M, N, K):
    A = draw(M, K, ("int", -4, 4), 3600 + M)
    B = draw(K, N, ("int", -4, 4), 3601 + M)
    dA, dB = upload(A), upload(B)
    for out, dtype in (("f32", torch.float32), ("bf16", torch.bfloat16), ("f32", torch.float32)):
        C = torch.full((M, N), float("nan"), dtype=dtype, device="cuda")
        sg().sfc_gemm_ex(dA, dB, C, ca_layers=0)
        assert np.array_equal(to_host(C), want_of(A, B, K, N, out)), (M, N, K, out)


def test_layers_on_two_streams():
    M, N, K = 16, 768, 16384
    ops = []
    for i in range(2):
        A, B = draw(M, K, ("int", -4, 4), 3700 + 2 * i), draw(K, N, ("int", -4, 4), 3701 + 2 * i)
        ops.append((upload(A), upload(B), want_of(A, B, K, N, "f32"), torch.cuda.Stream(),
                    [torch.full((M, N), float("nan"), device="cuda") for _ in range(4)]))
    torch.cuda.synchronize()
    for j in range(4):
        for dA, dB, _, s, Cs in ops:
            sg().sfc_gemm(dA, dB, Cs[j], ca_layers=0, stream=s)
    torch.cuda.synchronize()
    for _, _, want, _, Cs in ops:
        for C in Cs:
            assert np.array_equal(to_host(C), want)


# captured into a graph on a stream without library memory and on a stream that has
# it; replays beside eager work on the same operands give the eager result each time
@pytest.mark.parametrize("warm", [False, True])
def test_graph_capture(warm):
    M, N, K = 13, 1024, 16384
    A, B = draw(M, K, ("int", -4, 4), 3900), draw(K, N, ("int", -4, 4), 3901)
    dA, dB, want = upload(A), upload(B), want_of(A, B, K, N, "f32")
    C = torch.full((M, N), float("nan"), device="cuda")
    E = torch.full((M, N), float("nan"), device="cuda")
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        if warm:
            sg().sfc_gemm(dA, dB, E, ca_layers=0)
        g = torch.cuda.CUDAGraph()
        torch.cuda.synchronize()
        with torch.cuda.graph(g, stream=s):
            sg().sfc_gemm(dA, dB, C, ca_layers=0)
        for _ in range(3):
            C.fill_(float("nan"))
            g.replay()
            sg().sfc_gemm(dA, dB, E, ca_layers=0)
            torch.cuda.synchronize()
            assert np.array_equal(to_host(C), want)
            assert np.array_equal(to_host(E), want)
            E.fill_(float("nan"))


# operands whose sums depend on their order: a recorded call has the bits of the call
# that runs at once (and of the entry point that allocates nothing) on a cold and on a
# warm stream, also after a call that grows the stream's memory and on another stream
@pytest.mark.parametrize("warm", [False, True])
def test_graph_capture_keeps_the_bits(warm):
    M, N, K = 13, 1024, 16384
    dA, dB = upload(draw(M, K, ("normal", 0.0, 1.0), 3910)), upload(draw(K, N, ("normal", 0.0, 1.0), 3911))
    lA, lB = upload(draw(128, 65535, ("normal", 0.0, 1.0), 3912)), upload(draw(65535, 128, ("normal", 0.0, 1.0), 3913))
    want, got, large = (torch.empty(s, device="cuda") for s in ((M, N), (M, N), (128, 128)))
    sg().sfc_gemm_noalloc_ex(dA, dB, want, ca_layers=0)
    s, t = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(s):
        if warm:
            sg().sfc_gemm(dA, dB, got, ca_layers=0)
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            sg().sfc_gemm(dA, dB, got, ca_layers=0)
        eager = torch.empty_like(got)
        for replay_on in (s, t, s):
            got.fill_(float("nan"))
            sg().sfc_gemm(lA, lB, large, ca_layers=0)
            sg().sfc_gemm(dA, dB, eager, ca_layers=0)
            torch.cuda.synchronize()
            with torch.cuda.stream(replay_on):
                g.replay()
            torch.cuda.synchronize()
            assert torch.equal(got.view(torch.int32), want.view(torch.int32))
            assert torch.equal(eager.view(torch.int32), want.view(torch.int32))


# infinities and NaN stay in their rows and columns (a block's neighbours, and K
# past a ragged end, hold zeros and not other rows' values)
def test_special_values_stay():
    M, N, K = 21, 70, 45
    A = draw(M, K, ("int", 1, 4), 3800)
    B = draw(K, N, ("int", 1, 4), 3801)
    dA, dB = upload(A), upload(B)
    dA[3, K - 1], dA[5, 0], dB[K - 1, N - 1] = float("inf"), float("nan"), float("-inf")
    C = torch.empty((M, N), dtype=torch.float32, device="cuda")
    sg().sfc_gemm(dA, dB, C, ca_layers=1)
    ref = dA.double().cpu() @ dB.double().cpu()
    assert torch.equal(torch.nan_to_num(C.double().cpu(), nan=12345.0), torch.nan_to_num(ref, nan=12345.0))
