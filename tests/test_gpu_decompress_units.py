"""nm_decompress_i8 from the tiled layout: the kernel of whole units (aligned arrays) and the one of bytes (any other place) give the oracle's
integers, for every pattern, with row counts around the 16 of a block and block counts around the four of a workgroup."""
import numpy as np
import pytest
import torch

import oracle
import paper_2206_15014_amd as nm

pytestmark = pytest.mark.gpu

PATTERNS = [(1, 4), (2, 4), (3, 4), (4, 4)] + [(n, 8) for n in range(1, 9)]


def _at(offset, t):
    """A copy of the tensor whose first byte lies `offset` bytes behind an aligned address."""
    flat = torch.empty(offset + t.numel() + 16, dtype=t.dtype, device=t.device)[offset:offset + t.numel()]
    flat.copy_(t.reshape(-1))
    return flat.reshape(t.shape)


@pytest.mark.parametrize("N, M", PATTERNS)
@pytest.mark.parametrize("bits", [4, 8])
@pytest.mark.parametrize("rows, cols", [(1, 128), (16, 128), (17, 384), (47, 640), (80, 256)])
def test_units_and_bytes(N, M, bits, rows, cols):
    W = (np.random.default_rng(rows * cols + N).standard_normal((rows, cols)) * 0.02).astype(np.float32)
    v, m, _ = oracle.compress(W, N, M, bits)
    want = oracle.decompress(v, m, rows, cols, N, M, bits)
    vals, meta, _ = nm.nm_compress(torch.from_numpy(W).cuda(), N, M, bits, layout=nm.NM_LAYOUT_TILED)
    for v, m, o in ((0, 0, 0), (16, 16, 16), (8, 0, 0), (0, 2, 0), (0, 0, 4), (0, 0, 1)):
        out = _at(o, torch.full((rows, cols), 99, dtype=torch.int8, device="cuda"))
        nm.nm_decompress_i8(_at(v, vals), _at(m, meta), rows, cols, N, M, bits, out=out, layout=nm.NM_LAYOUT_TILED)
        assert np.array_equal(out.cpu().numpy(), want), (v, m, o)
