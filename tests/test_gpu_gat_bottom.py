"""Backward pass of the GAT's bottom layer at the edges of its tiles: entries of a destination around one and two tiles of
sixteen, widths around a block of sixteen features and around the bars of 128 and 192 where the kernel changes, heads that
are no power of two, and destinations without any source, against the oracle."""
import pytest

import workloads
from test_gpu_gat import _check, _dev, _run

pytestmark = pytest.mark.gpu

# fanout of the bottom layer (entries: one more), input width, heads
SHAPES = [(15, 100, 4), (16, 128, 4), (14, 132, 3), (31, 192, 8), (33, 12, 1), (17, 196, 2), (64, 64, 8), (3, 4, 5)]


@pytest.mark.parametrize("fan, width, heads", SHAPES)
def test_tiles_widths_and_heads(fan, width, heads):
    w = workloads.custom(3000, 240000, dims=[width, 4 * heads, 6], fanouts=[fan, 4], batch=333, n_splits=3, name="gat-bottom")
    _check(_run(w, [heads, 1], _dev(), seed=9, it=2), 2)


def test_fewer_sources_than_the_fanout():
    w = workloads.custom(9000, 18000, dims=[36, 16, 5], fanouts=[20, 6], batch=500, n_splits=2, name="gat-sparse")
    _check(_run(w, [4, 1], _dev(), seed=4, it=1), 2)
