"""Forms of the split products on both sides of each bar of their rules."""
import pytest

from split_rules import FEW, NARROW, WIDE, form, grad_block


# rows x K x N
@pytest.mark.parametrize("rows, K, N, want", [
    (32 * 32, 256, 256, FEW), (32 * 32 + 1, 256, 256, NARROW),              # 256 workgroups of 32 x 32
    (64 * 32, 260, 256, FEW), (64 * 32 + 1, 260, 256, NARROW),              # 512 from longer contractions on
    (64 * 192, 200, 256, NARROW), (64 * 192 + 1, 200, 256, WIDE),           # 768 narrow tiles, three per compute unit
    (10 ** 6, 200, 64, NARROW), (10 ** 6, 200, 65, WIDE),
    (10 ** 6, 200, 172, NARROW), (10 ** 6, 200, 193, WIDE),                 # less padding of the columns
])
def test_rows_in_pieces(rows, K, N, want):
    assert form(2 * rows, rows, K, N) == want


# A compute unit holds two workgroups, and a narrow tile costs nearly what a wide one costs: one per compute unit
# (6000 x 254 x 256: wide 12.8 us, narrow 16.0; 3300: 12.2, 10.4)
@pytest.mark.parametrize("rows, K, N, want", [
    (64 * 64, 254, 256, NARROW), (64 * 64 + 1, 254, 256, WIDE), (6000, 254, 256, WIDE), (11000, 202, 100, WIDE),
    (8192, 202, 100, NARROW), (8000, 70, 260, WIDE), (10 ** 6, 19, 140, WIDE), (10 ** 6, 19, 64, NARROW), (777, 254, 256, FEW),
])
def test_rows_float_by_float(rows, K, N, want):
    assert form(2 * rows, rows, K, N, pieces=False) == want


def test_heads_count_together():
    assert form(2000, 1000, 128, 64, heads=4) == FEW and form(2000, 1000, 128, 64, heads=8) == NARROW


def test_blocks_of_the_weight_gradients():
    assert grad_block(2 * 96 * 64, 512, 256) == 128 and grad_block(2 * 96 * 64 - 1, 512, 256) == 64
    assert grad_block(10 ** 6, 64, 256) == grad_block(10 ** 6, 256, 64) == 64
