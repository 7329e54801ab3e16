"""256-row tiles by the number of their 16-row blocks that hold rows: every number that the K loop is compiled for (0 to 8 for each
of the two rows of wavefronts), with a last block that is full, half full and of one row, beside slots of two, three and more
than eight tiles; every row compared.  Few tiles, K of two K tiles, of several, and with a tail; so many tiles that a workgroup walks
several with different numbers of blocks (each requests the next one's operands in its last two K tiles: from its start where
it has two, after one where it has three), and whose stores are still on their way in the next one's first K tile; and tiles cut
along K into four pieces, by the same numbers of blocks."""
import pytest

import paper_2503_06823_amd as P
from gpu_util import TILED, check_grouped_ffn, ffn_path

pytestmark = pytest.mark.gpu

WORKGROUPS = 256  # of the persistent launch


def slots(missing):
    return [16 * b - missing for b in range(1, 17)] + [0, 257, 272, 512 - missing, 515, 2049 + missing, 7000]


def tiles_and_pieces(rows, N, K, columns):
    """Output tiles of a product, and into how many pieces along K those that do not fill a round are cut."""
    tiles = sum(-(-r // 256) for r in rows) * -(-N // columns)
    left = tiles % WORKGROUPS
    return tiles, min(WORKGROUPS // left, max(-(-K // 64) // 8, 1), 8) if left else 1


@pytest.mark.parametrize("act", ["swiglu", "relu"])
@pytest.mark.parametrize("d,f", [(128, 128), (128, 392), (392, 256)])
@pytest.mark.parametrize("missing", [0, 7, 15])
def test_every_number_of_blocks(gpu_device, act, d, f, missing):
    rows = slots(missing)
    desc = P.make_desc(sum(rows), d, f, len(rows), 1, len(rows), "bf16", act)
    assert ffn_path(desc) == TILED
    check_grouped_ffn(desc, act, rows, 100 * missing + d + f, gpu_device)


@pytest.mark.parametrize("act", ["swiglu", "relu"])
# two K tiles, three with a tail, three whole ones in the product of many tiles; 37 K tiles with a tail and without in the one that is cut
@pytest.mark.parametrize("short,long", [(128, 2312), (136, 2368), (192, 2312)])
@pytest.mark.parametrize("first", ["many", "cut"])
@pytest.mark.parametrize("missing", [0, 7, 15])
def test_many_tiles_and_cut_ones(gpu_device, act, short, long, first, missing):
    rows = slots(missing)
    d, f = (short, long) if first == "many" else (long, short)
    desc = P.make_desc(sum(rows), d, f, len(rows), 1, len(rows), "bf16", act)
    assert ffn_path(desc) == TILED
    products = [tiles_and_pieces(rows, f, d, 128 if act == "swiglu" else 256), tiles_and_pieces(rows, d, f, 256)]
    many, cut = products if first == "many" else products[::-1]
    assert many[0] > 2 * WORKGROUPS and many[0] % WORKGROUPS
    assert cut[0] < WORKGROUPS and cut[1] >= 2
    check_grouped_ffn(desc, act, rows, 100 * missing + d + f, gpu_device)
