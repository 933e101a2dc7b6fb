"""How the planner cuts row pairs on the three-plane kernel, read off the workspace (host only): packed weights, and two partial
tiles for every block that shares tiles."""
from paper_1412_4564_amd import binding as B

UNIT = 3 * 3 * 2 * 128 * 16          # bytes of packed weights: 3 columns x 3 planes x 2 octets x 128 filters x 8 channels
TILE = 128 * 64 * 2 * 4              # bytes of a partial tile: 128 filters x 64 pairs of rows


def test_a_tile_of_row_pairs_is_cut_into_at_most_32_pieces():
    # 7 x 13 pairs of rows, two images: three tiles; 256 channels: 64 units
    d = B.make_desc((2, 256, 13, 14), (96, 256, 3, 3), (1, 1), (1, 1, 1, 1))
    assert B.mcn_conv_kernel_name(d, 0) == "igemm_f23"
    assert B.mcn_conv_workspace_size(d, 0) == 64 * UNIT + 2 * (3 * 32) * TILE


def test_enough_tiles_are_cut_for_every_compute_unit():
    # 7 x 14 pairs, one image: two tiles for each of four tiles of filters
    d = B.make_desc((1, 512, 14, 14), (512, 512, 3, 3), (1, 1), (1, 1, 1, 1))
    assert B.mcn_conv_workspace_size(d, 0) == 4 * 128 * UNIT + 2 * 256 * TILE
