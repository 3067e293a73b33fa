"""4-bit weights are multiplied as 16 times their value in the tiled-layout kernels: exact sums at the largest magnitudes the codes
have, on both sides of the reduction length up to which 16 times the sum fits 32 bits, and on either side of the lines between tiles."""
import numpy as np
import pytest
import torch

import oracle
import paper_2206_15014_amd as nm

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N, M", [(2, 4), (1, 4), (3, 4), (4, 4), (1, 8), (2, 8), (5, 8)])
@pytest.mark.parametrize("T, K, O", [(3, 128, 96), (40, 4096, 192), (700, 256, 768), (1100, 640, 1056)])
def test_extreme_codes(N, M, T, K, O):
    rng = np.random.default_rng(T + N)
    W = rng.choice(np.array([-1.0, 1.0], np.float32), (O, K))          # every kept code is -7 or 7
    W[0], W[1] = 1.0, -1.0                                             # the largest sums of either sign
    X = rng.choice(np.array([-128, 127], np.int8), (T, K))
    X[0], X[-1] = 127, -128
    v, m, s = oracle.compress(W, N, M, 4)
    want = oracle.gemm_sparse(X, v, m, O, N, M, 4)
    vals, meta, scales = nm.nm_compress(torch.from_numpy(W).cuda(), N, M, 4, layout=nm.NM_LAYOUT_TILED)
    acc = torch.empty((T, O), dtype=torch.int32, device="cuda")
    nm.nm_gemm(torch.from_numpy(X).cuda(), 1.0, vals, meta, scales, O, N, M, 4, acc=acc, layout=nm.NM_LAYOUT_TILED)
    assert np.array_equal(acc.cpu().numpy(), want)


# (2:4: K / 2 kept.)  131072 - 64 kept entries are the last whole slice below the limit, 131072 the first past it, whose products by -128
# and -8 would reach 2^31
@pytest.mark.parametrize("K", [2 * 131072 - 128, 2 * 131072])
def test_longest_reductions(K):
    T, O = 2, 16
    codes = np.full((O, K // 4), 0x88, np.uint8)                       # two codes of -8 a byte, on columns 0 and 1 of each group
    meta = np.full((O, K // 4 * 4 // 8), 0x44, np.uint8)
    X = np.full((T, K), -128, np.int8)
    X[1] = 127
    v, m = oracle.to_tiled(codes, meta, K, 2, 4, 4)
    acc = torch.empty((T, O), dtype=torch.int32, device="cuda")
    nm.nm_gemm(torch.from_numpy(X).cuda(), 1.0, torch.from_numpy(v).cuda(), torch.from_numpy(m).cuda(), torch.ones(O, device="cuda"), O, 2, 4, 4,
               acc=acc, layout=nm.NM_LAYOUT_TILED)
    want = np.array([[K // 2 * 8 * 128] * O, [K // 2 * -8 * 127] * O], np.int64)
    assert np.array_equal(acc.cpu().numpy().astype(np.int64), want)


# (One column of codes -8 a row against activations of -128 and 127.)  Past the few-token kernels' eight shares, and many tokens past
# the limit of one share: a tile that extends the signs
@pytest.mark.parametrize("N, M, T, K, O", [(2, 4, 2, 8 * 2047 * 128, 16), (2, 4, 2, 8 * 2047 * 128 + 128, 16), (2, 4, 2100, 2 * 131072, 256),
                                           (4, 4, 1030, 131072 + 128, 520), (1, 8, 140, 8 * 131072, 1040), (5, 8, 1030, 8 * 26240, 520)])
def test_longest_reductions_on_matrix_tiles(N, M, T, K, O):
    pieces = nm.nm_packed_sizes(O, K, N, M, 4, nm.NM_LAYOUT_TILED)
    vals = torch.full((pieces[0],), 0x88, dtype=torch.uint8, device="cuda")
    if M == 8 and N == 5:                                              # offsets 0 1 2 3 4 | 0 1 2 3 4: whole groups from the oracle's own packing
        W = np.tile(np.array([-7, -7, -7, -7, -7, 0, 0, 0], np.float32), (16, 128 // 8))
        _, m, _ = oracle.compress(W, N, M, 4)
        _, tiled = oracle.to_tiled(np.zeros((16, 128 // 8 * 5 // 2), np.uint8), m, 128, N, M, 4)
        meta = torch.from_numpy(np.tile(tiled.reshape(-1), pieces[1] // tiled.size)).cuda()
    else:
        meta = torch.full((max(pieces[1], 1),), {(2, 4): 0x44, (4, 4): 0, (1, 8): 0}[N, M], dtype=torch.uint8, device="cuda")
    X = torch.full((T, K), -128, dtype=torch.int8, device="cuda")
    X[1::2] = 127
    acc = torch.empty((T, O), dtype=torch.int32, device="cuda")
    nm.nm_gemm(X, 1.0, vals, meta, torch.ones(O, device="cuda"), O, N, M, 4, acc=acc, layout=nm.NM_LAYOUT_TILED)
    assert nm.binding.raw().nm_bench_last_gemm_tile() > 0
    kept = K // M * N
    assert torch.equal(acc[0::2], torch.full_like(acc[0::2], kept * 8 * 128)) and torch.equal(acc[1::2], torch.full_like(acc[1::2], -kept * 8 * 127))


# (kind of output, tile): one round and two, 128 and 96 columns, outputs written through and not, whole and ragged tiles, and the two-stage
# tiles of short reductions
@pytest.mark.parametrize("N, M", [(2, 4), (1, 4), (4, 4)])
@pytest.mark.parametrize("T, K, O, kind, tile", [
    (2750, 128, 576, "bf16", 115), (2750, 256, 640, "bf16", 127), (6010, 384, 768, "bf16", 115), (6010, 384, 576, "f32", 127), (16010, 128, 480, "bf16", 117),
    (9010, 256, 1024, "q8", 117), (7990, 384, 1024, "q8", 127), (9010, 256, 1024, "f32", 127), (12300, 256, 768, "bf16", 117), (24600, 128, 480, "q8", 115),
    (4100, 256, 2304, "bf16", 133), (700, 256, 768, "bf16", None)])
def test_exact_on_every_tile_of_the_rule(N, M, T, K, O, kind, tile):
    rng = np.random.default_rng(T + N + O)
    W = rng.choice(np.array([-1.0, 1.0], np.float32), (O, K))
    W[0], W[-1] = 1.0, -1.0
    vals, meta, scales = nm.nm_compress(torch.from_numpy(W).cuda(), N, M, 4, layout=nm.NM_LAYOUT_TILED)
    Wq = nm.nm_decompress_i8(vals, meta, O, K, N, M, 4, layout=nm.NM_LAYOUT_TILED)
    X = torch.from_numpy(rng.choice(np.array([-128, 127, 3], np.int8), (T, K))).cuda()
    want = (X.float() @ Wq.float().t().contiguous()).int()            # |sums| <= 384 * 7 * 128 < 2^24: exact in fp32
    out = torch.empty((T, O), dtype={"bf16": torch.bfloat16, "f32": torch.float32, "q8": torch.int8}[kind], device="cuda")
    acc = torch.empty((T, O), dtype=torch.int32, device="cuda")
    ones = torch.ones(O, device="cuda")
    for with_acc in (True, False):                                     # either way out of the tile
        a = acc if with_acc and kind != "q8" else None
        if kind == "q8":
            nm.nm_gemm_q8(X, 1.0, vals, meta, ones, O, N, M, 4, 4096.0, out, layout=nm.NM_LAYOUT_TILED)
            assert torch.equal(out, (want.float() / 4096.0).round().to(torch.int8))       # powers of two: one rounding here too
        else:
            nm.nm_gemm(X, 1.0, vals, meta, ones, O, N, M, 4, acc=a, out=out, out_dtype=2 if kind == "bf16" else 1, layout=nm.NM_LAYOUT_TILED)
            assert torch.equal(out, want.to(out.dtype))                # one rounding, to nearest even, of an exact sum
        if tile is not None:
            assert nm.binding.raw().nm_bench_last_gemm_tile() == tile
        if a is not None:
            assert torch.equal(a, want)
