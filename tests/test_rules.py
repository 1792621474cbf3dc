"""The rules that choose between two kernels, held against times of both on one MI355X: the rule has the faster one wherever they
differ by more than an eighth."""
import pytest

import rules

# rows of `products` products, `length` entries in every row of B, columns anywhere in `windows` windows of 16384: numeric stage in us
# with products one by one, and in tiles
HEAVY = [
    # windows, products, length, one by one, tiles
    (1, 15728, 16, 242, 297), (1, 56376, 16, 380, 480), (1, 222971, 16, 284, 389), (1, 58934, 64, 373, 308), (1, 277121, 64, 334, 205),
    (1, 284059, 95.7, 311, 209), (1, 290552, 190.9, 301, 240), (2, 15733, 16, 364, 647), (2, 223011, 16, 389, 710), (2, 15861, 32, 331, 409),
    (2, 257558, 32, 339, 450), (2, 284523, 95.9, 328, 274), (2, 287892, 127.8, 360, 275), (2, 287213, 255, 324, 255), (2, 24000, 2, 822, 1892),
    (2, 24000, 8, 622, 1048), (4, 56392, 16, 901, 1574), (4, 223041, 16, 649, 1370), (4, 257635, 32, 523, 842), (4, 270715, 48, 461, 625),
    (4, 277493, 64, 430, 532), (4, 59334, 95.9, 557, 644), (4, 287848, 255.5, 378, 321), (8, 56391, 16, 1752, 4001), (8, 58761, 48, 1258, 1778),
    (8, 59356, 96, 866, 1146), (8, 288433, 127.9, 561, 643), (16, 15736, 16, 501, 783), (16, 56398, 16, 1957, 4228), (16, 277669, 64, 1141, 1937),
    (16, 288160, 255.9, 613, 736), (16, 24000, 2, 1994, 4493), (16, 24000, 32, 1079, 1469), (32, 15736, 16, 735, 1018), (32, 56398, 16, 2333, 4851),
    (32, 15830, 256, 1.0, 0.93), (64, 24000, 8, 2713, 5268), (64, 24000, 32, 1671, 2274), (64, 15830, 256, 1.0, 0.88), (64, 15841, 512, 1.0, 0.85),
    (128, 15836, 32, 1.0, 1.68), (128, 15890, 96, 1.0, 1.48), (128, 15964, 128, 1.0, 1.17), (128, 293767, 512, 1026, 1626),
    # power-law matrices: mean products and length of the rows that go through windows
    (1, 10279, 95.8, 195, 164), (1, 15336, 226.6, 367, 304), (2, 18071, 313.9, 754, 625), (4, 22856, 424.3, 1899, 1531), (8, 28879, 569.1, 4769, 3950),
    (16, 39606, 758.3, 13017, 10808),
    # columns in blocks of 8000, 20 000 and 60 000
    (1.5, 100000, 100, 866, 764), (1.5, 150000, 300, 994, 861), (1.5, 60000, 30, 1352, 1496), (2.2, 150000, 300, 1157, 1034), (2.2, 60000, 30, 1615, 1906),
    (2.2, 400000, 1000, 1846, 1589), (4.7, 100000, 100, 1554, 1740), (4.7, 60000, 30, 2385, 2918), (4.7, 400000, 1000, 2450, 2190),
]


@pytest.mark.parametrize("windows, products, length, one_by_one, tiles", HEAVY)
def test_heavy_rows_go_the_faster_way(windows, products, length, one_by_one, tiles):
    chosen = tiles if rules.load().heavy_in_tiles(1000.0 * products, 1000.0, 1000.0 * products / length, windows) else one_by_one
    assert chosen <= 1.125 * min(one_by_one, tiles)


# columns, products of a row, length of the rows of B: a call for the sizes of the rows in us with products one by one, and in tiles
SYMBOLIC = [
    (65536, 6000, 2, 332, 503), (65536, 24000, 2, 434, 714), (65536, 24000, 4, 306, 415), (65536, 6000, 12, 194, 156), (65536, 6000, 16, 202, 141),
    (65536, 6000, 32, 199, 124), (65536, 24000, 16, 200, 159), (65536, 24000, 48, 179, 123), (262144, 24000, 2, 449, 713), (262144, 6000, 12, 193, 157),
    (524288, 24000, 4, 310, 509), (524288, 24000, 12, 190, 241), (524288, 100000, 8, 335, 450), (524288, 24000, 48, 186, 170), (1 << 20, 24000, 8, 262, 382),
    (1 << 20, 24000, 12, 190, 259), (1 << 20, 100000, 16, 312, 398), (1 << 20, 6000, 24, 226, 201), (1 << 20, 24000, 48, 182, 162), (1 << 22, 100000, 4, 994, 2406),
    (1 << 22, 100000, 8, 742, 1472), (1 << 22, 100000, 24, 671, 824), (1 << 22, 100000, 32, 564, 676),
]


@pytest.mark.parametrize("cols, products, length, one_by_one, tiles", SYMBOLIC)
def test_symbolic_rows_go_the_faster_way(cols, products, length, one_by_one, tiles):
    chosen = tiles if rules.load().symbolic_in_tiles(10 ** 6, cols, 1000 * products, 1000 * products // length) else one_by_one
    assert chosen <= 1.125 * min(one_by_one, tiles)


def test_no_tiles_of_a_matrix_smaller_than_what_a_lane_reads():
    assert not rules.load().symbolic_in_tiles(7, 1000, 10 ** 9, 1) and rules.load().symbolic_in_tiles(8, 1000, 10 ** 9, 1)


# products, the largest row's, a call for the sizes of the rows in us with the rows above 32768 products in a launch of larger
# workgroups, and with all rows in smaller ones (256 compute units)
FEW = [
    (44 * 10 ** 6, 4 * 10 ** 6, 394, 535), (406 * 10 ** 6, 4 * 10 ** 6, 604, 688), (375 * 10 ** 6, 1500000, 215, 280), (75 * 10 ** 6, 300000, 325, 343),
    (300 * 10 ** 6, 300000, 458, 416), (120 * 10 ** 6, 60000, 218, 196), (120 * 10 ** 6, 60000, 178, 164), (118 * 10 ** 6, 256000, 275, 244),
    (179 * 10 ** 6, 256000, 295, 267), (1136 * 10 ** 6, 17 * 10 ** 6, 818, 883), (3005 * 10 ** 6, 40 * 10 ** 6, 1664, 1980),
]


@pytest.mark.parametrize("products, largest, apart, together", FEW)
def test_rows_of_many_products_are_apart_where_that_is_faster(products, largest, apart, together):
    limit = rules.load().symbolic_few_products(products, largest, 256)
    assert limit in (32768, largest)
    assert (together if limit == largest else apart) <= 1.06 * min(apart, together)


# columns, entries of every row of B, 6 M entries in all: the stage with its sorted copy in us, by a network and by the bitmap
SORTED = [
    (32768, 300, 258, 244), (32768, 600, 281, 168), (32768, 3000, 455, 199), (65536, 300, 260, 254), (65536, 1000, 149, 117), (131072, 200, 249, 384),
    (131072, 600, 279, 191), (131072, 3000, 459, 212), (262144, 200, 255, 590), (262144, 300, 260, 420), (262144, 2000, 254, 190), (524288, 200, 249, 1020),
    (524288, 600, 279, 407), (524288, 1000, 152, 188), (524288, 3000, 465, 279), (1 << 20, 200, 256, 1918), (1 << 20, 1000, 153, 287), (1 << 20, 2000, 260, 341),
    (1 << 20, 3000, 463, 395),
]


@pytest.mark.parametrize("cols, length, network, bitmap", SORTED)
def test_rows_of_the_sorted_copy_go_the_faster_way(cols, length, network, bitmap):
    assert (bitmap if length >= rules.load().sort_bitmap_from(cols) else network) <= 1.125 * min(network, bitmap)


def test_no_bitmap_of_more_than_four_turns():
    assert rules.load().sort_bitmap_from((1 << 20) + 1) == 4097 and rules.load().sort_bitmap_from(1) == 129


# windows, entries of a row of B, numeric stage in us of rows of 3000 products hashed, and in windows
MIDDLE = [
    (1, 64, 683, 594), (1, 250, 691, 573), (1, 1000, 725, 573), (4, 64, 727, 596), (4, 250, 745, 583), (16, 64, 798, 624), (16, 250, 816, 602),
    (16, 1000, 847, 617), (32, 64, 847, 918), (32, 250, 856, 803), (32, 1000, 886, 799),
]


@pytest.mark.parametrize("windows, length, hashed, windowed", MIDDLE)
def test_middle_rows_go_the_faster_way(windows, length, hashed, windowed):
    assert (windowed if rules.load().middle_in_windows(windows, length * 1000, 1000) else hashed) <= 1.05 * min(hashed, windowed)
