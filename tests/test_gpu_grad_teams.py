"""Weight gradients in blocks of 128, which two teams of four waves form from every other 32 rows of a chunk and finish by
halves: chunks whose last 64 rows give the second team nothing, part of a step and a whole one, blocks whose lower half lies
outside the matrix, against float64 within the bound of a float32 sum; and values that only one of the teams meets and the
parts of a product cannot carry."""
import pytest
import torch

from split_rules import grad_block
from test_gpu_split_products import N_VERT, _case, _within

pytestmark = pytest.mark.gpu


# chunks of 96 rows (88 in the last one, 60), of 320 (185) and of 512 (288); with N = 129 of 96, 96, 416 and 640
@pytest.mark.parametrize("rows", [664, 1500, 12345, 19744])
@pytest.mark.parametrize("D, N", [(129, 255), (130, 200), (150, 200), (200, 129)])
def test_chunks_of_two_teams(rows, D, N):
    assert grad_block(N_VERT, 2 * D, N) == 128
    _, gw, gb, X, _, _, dz = _case(rows, D, N, N_VERT)
    _within(gw, X.T @ dz, X.abs().T @ dz.abs(), rows)
    _within(gb, dz.sum(0), dz.abs().sum(0), rows)


@pytest.mark.parametrize("row", [5, 40])        # of the first team and of the second
def test_infinity_in_rows_of_one_team(row):
    def glog(dev, cap):
        gen = torch.Generator(device=dev)
        gen.manual_seed(row)
        z = torch.randn(cap, 200, generator=gen, device=dev)
        z[row, 3] = float("inf")
        return z

    _, gw, gb, X, _, _, dz = _case(1500, 130, 200, N_VERT, glog=glog)
    rest = torch.arange(200, device=gw.device) != 3
    _within(gw[:, rest], X.T @ dz[:, rest], X.abs().T @ dz[:, rest].abs(), 1500)
    assert torch.equal(torch.sign(gw[:, 3]).double(), torch.sign(X[row])) and bool(torch.isinf(gw[:, 3]).all())
    assert float(gb[3]) == float("inf")
