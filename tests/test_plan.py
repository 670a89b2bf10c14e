"""CPU tests of the launch shapes (csrc/plan.h) over the range of the sizes."""
import pytest

from tests import plan_lib

LIMIT = 1 << 32  # workgroups times threads of a dimension stay below this


@pytest.mark.parametrize("nblk,bands,nv", [
    (1, 1, 1), (8, 6, 1), (489, 6, 16), (2051, 4096, 2), (1954, 4096, 256), (1 << 21, 6, 1), (40_000, 6, 256)])
def test_binning_grid(nblk, bands, nv):
    """Every (block, band, view) has a workgroup of its own, at sizes where one
    dimension would not hold them all too (a wide and a tall view: 4,096 bands)."""
    x, y, z = plan_lib.grid("bin_grid", nblk, bands, nv)
    assert x % 8 == 0 and nblk <= x < nblk + 8 and y == bands and z == nv
    assert x * plan_lib.load().bin_threads() < LIMIT and y <= 65535 and z <= 65535
    # block (i % 8) x / 8 + i / 8 of workgroup i: each block once
    if x <= 4096:
        assert sorted(i % 8 * (x // 8) + i // 8 for i in range(x)) == list(range(x))


@pytest.mark.parametrize("slots", [1, 83, 84, 85, 5000, 16_000_000, 84 << 22, (84 << 22) + 1, 1_409_286_144,
                                   1_409_286_145, 2_200_000_000, LIMIT - 1])
def test_pair_sum_grid(slots):
    """The (view, Gaussian)s of all rows of workgroups cover every slot, with
    less than one row too many, up to the largest slot count."""
    plan = plan_lib.load()
    x, y, z = plan_lib.grid("sum_grid", slots)
    per = plan.sum_waves() * plan.sum_per_wave()
    assert per == 84 and z == 1
    assert x * y * per >= slots and x * (y - 1) * per < slots
    assert x * plan.sum_waves() * 64 < LIMIT and y <= 65535
    if slots <= per << 22:
        assert (x, y) == ((slots + per - 1) // per, 1)


@pytest.mark.parametrize("tiles,views", [(1, 1), (64, 1), (104, 12), (920, 1), (3600, 1), (8160, 1), (60_000, 16),
                                         (129_600, 1), (129_600, 4), (16_777_216, 1), (16_777_216, 256), (65, 64)])
def test_binning_blocks(tiles, views):
    """Blocks grow before their number, the length of a column of the count
    matrix, passes 256 (one view
    in blocks of 1,024: 320) or the matrix 2^20 entries, and no workspace has less
    room than a smaller Gaussian count needs."""
    plan = plan_lib.load()
    room, largest = 0, (tiles + views - 1) // views
    for n in sorted([0, 1, 255, 256, 257, 4096, 30_011, 65_536, 65_537, 100_000, 131_073, 262_144, 300_007, 524_288, 524_289,
              1_000_000, 4_000_000, 100_000_000, LIMIT - 1] + list(range(2000, 6_000_000, 65_521))):
        chunk = plan.bin_chunk(n, views, tiles, largest)
        blocks = plan.bin_blocks(n, chunk)
        assert blocks * chunk >= n and chunk % plan.bin_threads() == 0
        # a wave's share of a block is counted in 16 bits, and so is the block's
        assert 256 <= chunk <= 16384
        if n <= 256 * 2048 and tiles <= 4096:
            assert blocks <= (320 if chunk == 1024 and views == 1 else 256) and blocks * tiles <= 1 << 20
        assert blocks * largest <= 12 << 20 or chunk == 4096  # nor a view's part 12 x 2^20 in blocks of less than 4,096
        here = plan.bin_matrix_room(n, tiles, largest)
        assert blocks * tiles <= here and here >= room
        room = here


def test_tags_of_a_splat():
    """The up to 64 pairs that a splat has in one step of the scatter (a piece
    of its rectangle, row by row) have tags of their own in a view of any width."""
    plan = plan_lib.load()
    for tiles_x in list(range(1, 700)) + list(range(1016, 1032)) + [2047, 2048, 2049, 4095, 4096]:
        pitch = plan.bin_tag_pitch(tiles_x)
        assert tiles_x <= pitch < tiles_x + 128
        for width in list(range(1, min(tiles_x, 64) + 1)) + ([tiles_x // 2 + 1, tiles_x] if tiles_x < 900 else []):
            assert plan.shared_tags(width, pitch) == 0, (tiles_x, pitch, width)
    # most views keep their own width
    assert all(plan.bin_tag_pitch(t) == t for t in (26, 40, 80, 120, 240)) and plan.bin_tag_pitch(256) > 256


@pytest.mark.parametrize("views", [[(1, 1)], [(8, 8)], [(120, 68)], [(4096, 3), (8, 4096)], [(4096, 4096)], [(1, 4096), (2, 5)],
                                   [(480, 270)], [(4096, 8), (8, 4096)], [(16, 9), (240, 135)]])
def test_binning_bands(views):
    """A band fits the scatter's LDS (12 bytes a tile beside 5,136 bytes of
    marks, tags and sums, 64 KB in all), and is as high as its own view's width
    allows up to a sixth of the tallest view's rows."""
    plan = plan_lib.load()
    tallest = max(ty for _, ty in views)
    for tx, ty in views:
        rows = plan.bin_rows(tx, tallest)
        assert rows >= 1 and 12 * rows * tx + 5136 <= 65536
        assert rows == (tallest + 5) // 6 or (rows + 1) * tx > 4864


@pytest.mark.parametrize("sizes,forms", [
    ([(17, 9)], ["tiles"]), ([(640, 360)], ["tiles"]), ([(640, 705)], ["tiles"]), ([(400, 300)] * 4, ["tiles"]),
    ([(705, 700)], ["strips"]), ([(960, 540)], ["strips"]), ([(97, 4700)], ["tiles"]), ([(800, 720)], ["tiles"]),
    ([(1280, 720)], ["strips"]), ([(1920, 1080)], ["strips"]), ([(400, 300)] * 16, ["strips"]),
    # many small views: what one launch holds decides, not all pixels
    ([(300, 100)] * 17, ["strips", "tiles"]), ([(128, 128)] * 28, ["tiles"] * 2), ([(64, 64)] * 130, ["tiles"] * 9),
    ([(64, 64)] * 256, ["tiles"] * 16), ([(1920, 1080)] + [(64, 64)] * 16, ["strips", "tiles"]),
    # strips badly filled
    ([(65, 20_000)], ["tiles"]), ([(32_767, 20)], ["tiles"])])
def test_form_of_the_loss(sizes, forms):
    assert plan_lib.loss_forms(sizes) == forms


def test_shares_of_strips_fit_the_room_of_tiles():
    """The workspace holds one share per 16 x 16 tile and channel; strips are
    taken only where they are fewer, whatever the views' sizes."""
    for w in list(range(1, 70)) + [127, 128, 129, 255, 700, 1920, 32_767]:
        for h in [1, 2, 33, 34, 35, 68, 69, 500, 5000, 32_767]:
            tiles, strips = -(-w // 16) * -(-h // 16), -(-w // 64) * -(-h // 34)
            assert not plan_lib.load().loss_in_strips(tiles, strips, w * h) or strips <= tiles
