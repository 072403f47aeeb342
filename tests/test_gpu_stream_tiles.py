"""65..256 rows in the tiles with fewer activation lines to each weight line (96 x 128, and 96, 128, 192, 256 x 256) at the edges of their rows, logits
included, against at most 64 rows at a time.  Which product takes which of them is pinned in test_stream_tiles.py."""
import pytest

import eagle3_synth as S
from test_gpu_row_tiles import FEW, _rows_alone_and_together

pytestmark = pytest.mark.gpu


# 8B width: split and staggered 96 x 128 tiles, the LM head staggered and 256 weight rows wide; "wide": the same in step, gate/up 256 wide, a LM head
# that ends within a tile.  First, last and one more than the last row of 96, 128, 192 and 256, and a half and a whole row block of 32
@pytest.mark.parametrize("name", ["8b", "wide"])
@pytest.mark.parametrize("B,N,group", [(65, 1, 64), (80, 1, 40), (19, 5, 12), (96, 1, 64), (97, 1, 49), (127, 1, 64), (191, 1, 64), (64, 3, 21), (193, 1, 61), (51, 5, 12)])
def test_rows_in_tiles_with_few_activation_lines(name, B, N, group):
    _rows_alone_and_together(FEW[name], B, N, group, logits=True)


# 96 x 128 in five ranges and unsplit with a LM head that ends within a tile; down in eight ranges of 192 x 256 tiles
@pytest.mark.parametrize("B,N,group", [(90, 1, 60), (180, 1, 60)])
def test_rows_in_split_tiles(B, N, group):
    full = S.get_shape("c3").with_(name="split", hidden=5120, n_heads=40, n_kv_heads=8, intermediate=17408, vocab=20484)
    _rows_alone_and_together(full, B, N, group, logits=True)
