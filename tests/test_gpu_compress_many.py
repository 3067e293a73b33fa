"""nm_compress_batch of more than sixteen matrices and 32 MB, which goes out in launches of up to 48 with two shares of rows per
workgroup: the same bytes as nm_compress, matrix by matrix."""
import pytest
import torch

import paper_2206_15014_amd as nm

pytestmark = pytest.mark.gpu


# (count, rows, cols): 17 and 49 matrices (one past a launch), odd row counts (half-empty last workgroups, padded blocks of the tiled
# layout), one to four passes per wavefront on one, two and four wavefronts per row, widths that end inside a pass, mixed widths
SHAPES = [((17, 517, 1024),), ((49, 331, 768),), ((20, 150, 4096), (3, 1, 128)), ((18, 161, 3072), (5, 33, 1408), (1, 2, 2048)),
          ((40, 1000, 256), (9, 3, 4096))]


@pytest.mark.parametrize("scheme", [(2, 4, 8), (1, 4, 4), (4, 4, 4), (2, 8, 4), (1, 8, 8)])
@pytest.mark.parametrize("layout", [nm.NM_LAYOUT_ROWS, nm.NM_LAYOUT_TILED])
@pytest.mark.parametrize("shapes", SHAPES)
def test_many_matrices_as_one_by_one(shapes, layout, scheme):
    gen = torch.Generator(device="cuda").manual_seed(5)
    Ws = [torch.randn(rows, cols, device="cuda", generator=gen) * 0.02 for count, rows, cols in shapes for _ in range(count)]
    Ws[1][0].zero_()                           # a zero row, and a scale beyond the reciprocal's range
    Ws[2][0] *= 1e20
    assert sum(W.numel() for W in Ws) * 4 > 32 << 20 and len(Ws) > 16
    outs = nm.nm_compress_batch(Ws, *scheme, layout=layout)
    for W, got in zip(Ws, outs):
        for a, b in zip(got, nm.nm_compress(W, *scheme, layout=layout)):
            assert torch.equal(a, b)
