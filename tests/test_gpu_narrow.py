"""The kernels for rows of at most 16 channels (forward pass and feature gradient), where they can go wrong: every way a
row's width splits into loads, both depths of the packed parameters, clouds around one tile, K around the rows under way,
output blocks that reach past the width, hub points and empty lists, several clouds, both layouts."""
import pytest

import paper_1803_07289_amd as fx
from test_gpu_tile import check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("layout", [fx.BNC, fx.BCN], ids=["bnc", "bcn"])
@pytest.mark.parametrize("B,N,K,Din,Dout", [
    (1, 1, 1, 1, 16), (1, 63, 3, 2, 2), (1, 64, 4, 3, 64), (2, 65, 5, 4, 65), (3, 130, 7, 5, 130), (1, 97, 8, 6, 64),
    (1, 200, 9, 7, 12), (2, 129, 16, 8, 8), (1, 300, 17, 9, 64), (1, 90, 8, 10, 11), (1, 64, 12, 11, 70),
    (2, 70, 8, 13, 15), (1, 191, 8, 14, 16), (1, 500, 6, 16, 9), (1, 80, 8, 9, 300), (1, 80, 8, 70, 13),
    (1, 4097, 8, 64, 9), (2, 9000, 8, 9, 64),
])
def test_widths_and_sizes(B, N, K, Din, Dout, layout):
    check(30 + N + K, B, N, K, Din, Dout, layout)


def test_hub_point_and_empty_lists():
    check(5, 1, 500, 4, 9, 13, fx.BNC, hub=True)
    check(6, 2, 90, 8, 16, 4, fx.BCN, hub=True)
