"""What nm_gemm would launch in the tiled layout, read back without a GPU: where the tiles of a launch start on their walk along K."""
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
