"""The kernels for rows of at most 16 channels (forward pass and feature gradient), where they can go wrong: every way a
row's width splits into loads, both depths of the packed parameters, clouds around one tile, K around the rows under way,
output blocks that reach past the width, hub points and empty lists, several clouds, both layouts."""
import numpy as np
import pytest

import paper_1803_07289_amd as fx
from gpu_util import dev, from_layout, say, to_layout
from test_gpu_parity import random_problem
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


# point-major: the waves pack the parameters themselves; channel-major: the preparation launch does, beside turning the rows round
@pytest.mark.parametrize("Din,Dout", [(1, 1), (3, 32), (7, 65), (8, 64), (9, 64), (9, 13), (12, 130), (15, 3), (16, 200)])
def test_parameters_packed_by_the_waves_are_the_same_bits(Din, Dout):
    B, N, K = 2, 150, 5
    say(f"narrow, own parameters {Din}->{Dout}")
    pos, nbr, feat, theta, bias, _ = random_problem(30 + Din, B, N, K, Din, Dout)
    theta *= np.float32(2.0) ** np.random.default_rng(Din).integers(-40, 40, size=(3, Din, Dout)).astype(np.float32)
    theta[1, Din // 2] = 0
    bias[:, Dout // 2] = 0
    for bad in (None, np.inf):
        if bad is not None:
            theta[0, 0, Dout - 1] = bad
        out = [from_layout(fx.flexconv_fwd(to_layout(feat, layout), dev(pos), dev(nbr), dev(theta), dev(bias), layout=layout), layout)
               for layout in (fx.BNC, fx.BCN)]
        bits = [np.ascontiguousarray(o).view(np.uint32) for o in out]
        same = (bits[0] == bits[1]) | (np.isnan(out[0]) & np.isnan(out[1]))
        assert same.all()
