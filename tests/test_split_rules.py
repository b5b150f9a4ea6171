"""Forms of the split products on both sides of each bar of their rules."""
import pytest

import test_gpu_split_products as products
from split_rules import FEW, N_CU, NARROW, WIDE, form, grad_block, grad_chunks


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


def test_chunks_of_the_weight_gradients_fill_the_chip():
    """Blocks of 128, one workgroup a compute unit (two teams, that is two sums of rows a chunk), over all widths up to 1024:
    what a compute unit has to walk and the rows of a sum are no more than with one team a workgroup, two of them a compute
    unit and chunks in eights."""
    for tm in range(1, 17):
        for tn in range(1, 9):
            M, N, tiles = 128 * tm, 128 * tn, tm * tn
            assert grad_block(10 ** 7, M, N) == 128
            chunks, eights = grad_chunks(10 ** 7, M, N), max(8, 2 * N_CU // tiles // 8 * 8)
            rounds = -(-chunks * tiles // N_CU)
            assert rounds / chunks <= -(-eights * tiles // N_CU) / eights, (M, N)
            assert 2 * chunks >= eights, (M, N)
            assert 4 * tiles > N_CU or (rounds == 1 and chunks * tiles > N_CU - tiles), (M, N)
    assert [grad_chunks(10 ** 7, M, N) for M, N in ((1204, 256), (768, 384), (768, 256), (512, 256))] == [12, 14, 21, 32]
    assert grad_chunks(10 ** 7, 100, 132, 4) == 32 and grad_chunks(1000, 512, 256) == 32 and grad_chunks(1000, 1204, 1024) == 8


def test_products_at_the_edges_reach_every_form():
    """The shapes of test_gpu_split_products.py: forms x rows in pieces or float by float, and both blocks."""
    every = {(f, v) for f in (FEW, NARROW, WIDE) for v in (True, False)}

    def forms(shapes):
        return {(form(max(cap, r), r, 2 * D, N), D % 2 == 0) for cap in (1024, products.N_VERT) for r, D, N in shapes}

    def blocks(shapes):
        return {grad_block(max(cap, r), 2 * D, N) for cap in (1024, products.N_VERT) for r, D, N in shapes}
    assert forms([s[1:] for s in products.PRODUCTS]) == every
    assert {(grad_block(cap, 2 * D, N), D % 2 == 0, N % 4 == 0) for cap, r, D, N in products.PRODUCTS} == {
        (b, vx, vz) for b in (64, 128) for vx in (True, False) for vz in (True, False)}
    small, values = products.SMALL_OPERANDS, [(r, D, N) for r, N, D in products.VALUES]
    assert {f for f, _ in forms(small)} == {f for f, _ in forms(values)} == {FEW, NARROW, WIDE}
    assert {(WIDE, True), (WIDE, False)} <= forms(small) & forms(values)
    assert blocks(small) == blocks(values) == {64, 128}
    # contractions of one and two products: a wide tile, and blocks of 128
    assert form(products.N_VERT, 9000, 2, 200) == WIDE and grad_block(products.N_VERT, 260, 200) == 128
