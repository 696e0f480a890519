"""The convolution with room for packed point locations behind its workspace (flexconv_workspace_bytes_best) against the
same call in a workspace of the smallest size, which reads the location tensor itself: the same bits, and both within the
oracle's tolerance."""
import pytest
import torch

import oracle
import paper_1803_07289_amd as fx
from gpu_util import CANARY_BYTES, TOL, ExactWorkspace, dev, to_layout, from_layout, say
from helpers import rel_err
from test_gpu_parity import random_problem

pytestmark = pytest.mark.gpu


class BestWorkspace(ExactWorkspace):
    def __init__(self, op, B, N, K, Din, Dout, layout):
        self.need = int(fx.lib().flexconv_workspace_bytes_best(op, B, N, K, Din, Dout, layout))
        assert self.need >= fx.workspace_bytes(op, B, N, K, Din, Dout, layout) + 16 * B * N
        self.buf = torch.empty(self.need + CANARY_BYTES, dtype=torch.uint8, device="cuda")
        self.buf[self.need:] = 0xA5
        self.ws = self.buf[:self.need]


# clouds around a tile of 32 / 48 points and around a packing block of 2048, K around a batch of eight, several clouds;
# gathered widths of one lane group per row (64) and of half a one (32), in both directions
@pytest.mark.parametrize("layout", [fx.BNC, fx.BCN], ids=["bnc", "bcn"])
@pytest.mark.parametrize("B,N,K,Din,Dout", [
    (1, 1, 1, 64, 64), (2, 47, 8, 64, 64), (1, 49, 9, 64, 64), (3, 97, 16, 64, 64), (1, 2049, 5, 64, 64),
    (2, 33, 3, 64, 128), (1, 300, 8, 64, 32), (1, 300, 12, 32, 64), (2, 2047, 8, 32, 32),
])
def test_packed_locations_change_no_bit(B, N, K, Din, Dout, layout):
    say(f"packed locations: B={B} N={N} K={K} {Din}->{Dout} layout={layout}")
    pos, nbr, feat, theta, bias, g = random_problem(40 + N + K, B, N, K, Din, Dout)
    a = (to_layout(feat, layout), dev(pos), dev(nbr), dev(theta), dev(bias))
    gd = to_layout(g, layout)
    edges = fx.flex_inedges_build(a[2])
    results = []
    for kind in (ExactWorkspace, BestWorkspace):
        wf, wb = (kind(op, B, N, K, Din, Dout, layout) if op == fx.OP_CONV_FWD or Dout <= 64 else None
                  for op in (fx.OP_CONV_FWD, fx.OP_CONV_BWD))
        r = [fx.flexconv_fwd(*a, layout=layout, workspace=wf.ws)]
        if wb is not None:                   # (rows wider than 64 channels read the tensor either way)
            r += fx.flexconv_bwd(*a, gd, layout=layout, in_edges=edges, workspace=wb.ws)
            wb.check()
        wf.check()
        results.append(r)
    for x, y in zip(*results):
        assert torch.equal(x, y)
    assert rel_err(from_layout(results[1][0], layout), oracle.flexconv_fwd(feat, pos, nbr, theta, bias)) <= TOL
