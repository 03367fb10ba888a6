"""The any-alignment path (16-byte loads at element alignment into the LDS ring,
a ragged last K block through registers): the ends of rows, where a chunk is
loaded early and shifted, the last rows, the last K block of a layer, and the
limits where the path begins and ends.  Integer operands make every sum exact in fp32 (|sum| <= 16 K < 2^24), so
results are compared bit for bit; padding holds NaN, so an element used from
outside a row shows."""
import numpy as np
import pytest
import torch

from oracle import bf16 as obf16
from paper_2601_16294_amd.inputs import draw
from gpu_util import run_gemm, to_host, upload, sg

pytestmark = pytest.mark.gpu

TILES = ["128x128", "256x128", "128x256", "256x256"]


def check(M, N, K, tile, c, out, lda, ldb, ldc, seed):
    A = draw(M, K, ("int", -4, 4), seed, lda)
    B = draw(K, N, ("int", -4, 4), seed + 1, ldb)
    C = run_gemm(A, B, M, N, K, out=out, ldc=ldc, ca_layers=c, tile=tile)
    want = (obf16.bf16_to_f64(A[:, :K]).astype(np.int64) @ obf16.bf16_to_f64(B[:, :N]).astype(np.int64))
    want = want.astype(np.float32)
    if out == "bf16":
        want = obf16.bf16_to_f64(obf16.f32_to_bf16_rne(want))
    assert np.array_equal(C[:, :N], want.astype(np.float64)), (M, N, K, tile, c, out)
    assert np.isnan(C[:, N:]).all()


# every remainder of K and of N modulo the 8-element chunk, around the 64-deep
# block and the 128/256-wide tile
@pytest.mark.parametrize("r", range(8))
@pytest.mark.parametrize("tile", TILES)
def test_row_end_remainders(r, tile):
    check(129, 256 + r, 64 + r, tile, 1, "f32", 64 + r + 1, 256 + r + 3, 256 + r + 1, 2000 + r)
    check(131, 127 + r, 121 + r, tile, 2, "bf16", 121 + r, 127 + r, 127 + r, 2100 + r)


# the smallest sizes of the path, sizes below it (element loads), one row, one
# block column with fewer than 8 columns in the last chunk
@pytest.mark.parametrize("M,N,K", [(1, 8, 8), (3, 9, 15), (1, 1001, 77), (257, 8, 63), (65, 265, 9), (5, 7, 64),
                                   (64, 64, 7), (300, 513, 129)])
@pytest.mark.parametrize("tile", TILES)
def test_small_and_edge_sizes(M, N, K, tile):
    check(M, N, K, tile, 1, "f32", K + 1, N + 1, N, 2200 + M + N + K)
    check(M, N, K, tile, 1, "bf16", K, N, N + 5, 2300 + M + N + K)


# layers whose last blocks are whole and whose last layer runs past K
@pytest.mark.parametrize("c", [1, 2, 3, 7])
def test_layers(c):
    for K in (447, 448 + 1, 65):
        check(140, 261, K, "auto", c, "f32", K, 261, 261, 2400 + K + c)


def test_leading_dimension_limit():
    # 2^20 - 1 is the last leading dimension of A the ring's 32-bit offsets take
    for lda in ((1 << 20) - 1, 1 << 20, (1 << 22) - 1, 1 << 22):
        M, N, K = 3, 40, 72
        A = draw(M, K, ("int", -4, 4), 2500)
        B = draw(K, N, ("int", -4, 4), 2501)
        big = torch.full((M, lda), float("nan"), dtype=torch.bfloat16, device="cuda")
        big[:, :K] = upload(A)
        C = torch.empty((M, N), dtype=torch.float32, device="cuda")
        sg().sfc_gemm_ex(big[:, :K], upload(B), C)
        want = obf16.bf16_to_f64(A).astype(np.int64) @ obf16.bf16_to_f64(B).astype(np.int64)
        assert np.array_equal(to_host(C), want.astype(np.float64)), lda


# a last round of half-height blocks (a strip of block columns of its own), whose
# last columns may be fewer than the 8 that a shifted chunk needs
@pytest.mark.parametrize("N", [256 * 65 - 255, 256 * 65 - 250, 256 * 65 - 1])
def test_half_height_strip(N):
    check(1021, N, 77, "auto", 1, "f32", 77, N, N, 2600)


# aligned operands: the rows and columns of edge blocks, stored 16 bytes at a time
# where C's rows are aligned, and nothing outside C
@pytest.mark.parametrize("M,N", [(1, 8), (17, 120), (127, 136), (129, 248), (255, 264), (257, 504), (300, 256), (256, 520)])
@pytest.mark.parametrize("tile", TILES)
def test_edge_blocks_of_aligned_operands(M, N, tile):
    for out, pad in (("f32", 4), ("bf16", 8), ("f32", 1), ("bf16", 3)):
        check(M, N, 136, tile, 1, out, 136, N, N + pad, 2700 + M)
    check(M, N, 136, tile, 2, "f32", 136, N + 8, N, 2800 + M)


# leading dimensions of C around the limit of the edge stores' 32-bit offsets: rows
# inside C only, nothing right of C
@pytest.mark.parametrize("out", ["f32", "bf16"])
@pytest.mark.parametrize("ldc", [(1 << 22) - 8, 1 << 22])
def test_wide_rows_of_c(out, ldc):
    M, N, K = 131, 264, 72
    A, B = draw(M, K, ("int", -4, 4), 2900), draw(K, N, ("int", -4, 4), 2901)
    want = (obf16.bf16_to_f64(A) @ obf16.bf16_to_f64(B)).astype(np.float32)
    if out == "bf16":
        want = obf16.bf16_to_f64(obf16.f32_to_bf16_rne(want))
    C = torch.empty((M, ldc), dtype=torch.float32 if out == "f32" else torch.bfloat16, device="cuda")
    for tile in TILES:
        C[:, :N + 64] = float("nan")
        C[:, -64:] = float("nan")
        sg().sfc_gemm_ex(upload(A), upload(B), C[:, :N], tile=tile)
        assert np.array_equal(to_host(C[:, :N]), want.astype(np.float64)), tile
        assert torch.isnan(C[:, N:N + 64]).all() and torch.isnan(C[:, -64:]).all(), tile


# few rows in the last row of blocks, and layer copies (stored at device scope when
# the launch sums them itself)
@pytest.mark.parametrize("M", [1, 31, 32, 33, 129, 160, 161, 257, 290])
@pytest.mark.parametrize("tile", TILES)
def test_few_rows_in_the_last_blocks(M, tile):
    N, K = 328, 136
    for out in ("f32", "bf16"):
        check(M, N, K, tile, 1, out, K, N, N + 8, 2910 + M)
    A, B = draw(M, K, ("int", -4, 4), 2920), draw(K, N, ("int", -4, 4), 2921)
    C = torch.full((M, N), float("nan"), dtype=torch.float32, device="cuda")
    sg().sfc_gemm_fused_ex(upload(A), upload(B), C, ca_layers=3, tile=tile)
    want = obf16.bf16_to_f64(A) @ obf16.bf16_to_f64(B)
    assert np.array_equal(to_host(C), want)


# element loads (rows of fewer than 8 elements, leading dimensions past the ring's 32-bit
# offsets): several K blocks, a ragged last one, layers, every block shape
@pytest.mark.parametrize("tile", TILES)
@pytest.mark.parametrize("c", [1, 3])
def test_element_loads(tile, c):
    for M, N, K in ((300, 7, 520), (129, 3, 321), (270, 300, 7)):
        check(M, N, K, tile, c, "f32", K + 1, N, N + 1, 2950 + N)
        check(M, N, K, tile, c, "bf16", K, N + 2, N, 2960 + N)
    M, N, K = 140, 264, 457
    A, B = draw(M, K, ("int", -4, 4), 2970), draw(K, N, ("int", -4, 4), 2971)
    big = torch.full((M, 1 << 20), float("nan"), dtype=torch.bfloat16, device="cuda")
    big[:, :K] = upload(A)
    C = torch.full((M, N), float("nan"), dtype=torch.float32, device="cuda")
    sg().sfc_gemm_ex(big[:, :K], upload(B), C, ca_layers=c, tile=tile)
    want = obf16.bf16_to_f64(A) @ obf16.bf16_to_f64(B)
    assert np.array_equal(to_host(C), want)
