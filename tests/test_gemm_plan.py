"""What nm_gemm would launch in the tiled layout, read back without a GPU: the tile of narrow 4-bit layers, and where the tiles of a
launch start on their walk along K."""
import ctypes

import pytest

from paper_2206_15014_amd import binding

F32, BF16, CODES = 1, 2, 3


def plan(tokens, K, O, scheme, out=BF16):
    """(tile id, K blocks a token row starts behind the one before it, K blocks a column tile starts before the one before it)"""
    starts, (pattern, bits) = ctypes.c_int(-1), scheme.split("/")
    n, m = pattern.split(":")
    tile = binding.raw().nm_test_gemm_plan(tokens, K, O, int(n), int(m), int(bits), out, ctypes.byref(starts))
    blocks = K // (256 if tile == 113 else 128)
    return tile, starts.value >> 16, -(starts.value & 0xFFFF) % blocks


@pytest.mark.parametrize("tokens, K, O, scheme, want", [
    # one round: together, but on the two tiles that gain from HBM without a loss in the last-level cache
    (4096, 768, 768, "2:4/8", (116, 0, 0)), (8192, 3072, 768, "2:4/8", (112, 0, 0)), (2048, 1024, 1024, "2:4/8", (116, 0, 0)),
    (4096, 4096, 1024, "2:4/4", (127, 0, 0)), (4096, 3072, 768, "1:4/8", (115, 0, 1)), (3001, 3072, 768, "2:4/8", (113, 0, 2)),
    # several rounds, a CU to itself: one block, and three where one loses
    (49152, 4096, 1024, "2:4/8", (123, 1, 1)), (49152, 1024, 4096, "2:4/8", (123, 1, 1)), (24576, 2560, 640, "2:4/8", (121, 1, 3)),
    (49152, 2560, 640, "2:4/8", (128, 1, 3)), (49152, 1536, 384, "1:4/8", (122, 1, 1)),
    # two-stage tiles
    (24576, 1024, 3072, "2:4/8", (136, 1, 3)), (24576, 1024, 4096, "1:4/8", (133, 1, 1)), (24576, 768, 3072, "4:4/4", (133, 0, 1)),
    (128, 768, 768, "2:4/8", (143, 0, 0)),                  # few tokens: no such walk
])
def test_starts_along_k(tokens, K, O, scheme, want):
    assert plan(tokens, K, O, scheme) == want


def test_starts_are_the_launchs_own():
    """The distances are taken modulo the number of blocks, down to a single one."""
    for K in (128, 256, 384):
        tile, row, column = plan(49152, K, 1024, "2:4/8")
        assert 0 <= row < K // 128 and 0 <= column < K // 128


@pytest.mark.parametrize("tokens, K, O, out, tile", [
    # one round: 128 columns by eight wavefronts side by side where they divide the width, 128 x 96 where 96 alone does
    (4096, 768, 768, BF16, 127), (4096, 3072, 768, CODES, 127), (8192, 768, 384, BF16, 127), (4096, 768, 576, BF16, 115), (5000, 768, 480, F32, 115),
    # 96 columns take no more rounds than 128 / one more
    (6000, 384, 768, BF16, 115), (8192, 3072, 768, F32, 115), (5000, 768, 768, BF16, 127), (6000, 384, 576, BF16, 127), (9000, 768, 768, CODES, 127),
    (12288, 768, 576, BF16, 127), (24576, 768, 768, F32, 115),
    # written through (16-bit outputs from 14 MB, codes from 8): 128 x 128 by 4 x 2 wavefronts up to K = 2048, but where 96 is as good
    (8192, 384, 1024, CODES, 117), (8192, 2048, 896, BF16, 117), (12288, 1024, 640, BF16, 117), (12288, 1024, 640, CODES, 127), (8191, 384, 1024, CODES, 127),
    (8192, 2176, 1024, BF16, 127), (16000, 768, 768, BF16, 117), (12288, 640, 768, BF16, 117), (12288, 768, 768, BF16, 115), (16000, 3072, 768, BF16, 115),
    (24576, 768, 480, CODES, 115),
    # fp32 is always written through, sixteen columns at a time as well as any: never 117
    (24576, 384, 1024, F32, 127), (12288, 768, 640, F32, 127),
])
@pytest.mark.parametrize("scheme", ["2:4/4", "1:4/4", "4:4/4"])
def test_tile_of_narrow_4_bit_layers(tokens, K, O, out, tile, scheme):
    assert plan(tokens, K, O, scheme, out)[0] == tile


@pytest.mark.parametrize("K, few", [
    (2 * 131072 - 128, True), (2 * 131072, True),           # a wavefront of the few-token kernels walks an eighth of the reduction
    (8 * 2047 * 128, True), (8 * 2047 * 128 + 128, False),  # ... and 131072 kept entries from here on
])
def test_longest_4_bit_reductions_stay_on_matrix_tiles(K, few):
    assert plan(300, K, 768, "2:4/4")[0] == (142 if few else 127)
    assert plan(2, K, 16, "2:4/4")[0] == (141 if few else 127)
    assert plan(2048, K, 1024, "2:4/4")[0] == 127 and plan(2048, K, 1024, "4:4/4")[0] == 127      # (2048 rows of X: its offsets are 32 bits wide)
