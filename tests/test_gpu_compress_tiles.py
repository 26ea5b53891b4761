"""gqla_compress_cache at the edges between its ways of sharing the work out: up to 64 tiles of 128 tokens a workgroup takes a
quarter of a tile's latent dims, up to 96 a half, beyond it whole tiles.  Sequences with token counts around the halves and tiles, against the
fp64 product as in test_gpu_compress."""
import pytest

from test_gpu_compress import EDGES, test_compress_edges as check_compress

pytestmark = pytest.mark.gpu

SIX = EDGES * 6                                           # 114 tiles, 72 sequences


@pytest.mark.parametrize("g,d_h,d_v,lens", [
    (4, 128, 128, EDGES * 3 + [128 * 7]),                 # 64 tiles: quarters
    (4, 128, 128, EDGES * 3 + [128 * 7 + 1]),             # 65: halves
    (4, 128, 128, EDGES * 5 + [128]),                     # 96: halves
    (4, 128, 128, EDGES * 5 + [129]),                     # 97: whole tiles
    (3, 192, 256, SIX + [128 * 13, 300]),                 # 130: whole tiles, nine stages
    (8, 128, 128, [2000]),                                # 16 tiles, sixteen stages: the ring of quarters wraps
    (8, 128, 128, [128 * 70 - 1]),                        # 70 tiles: that of halves
])
def test_tiles(g, d_h, d_v, lens):
    check_compress(g, d_h, d_v, lens, 64, True)
