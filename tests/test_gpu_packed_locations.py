"""The convolution with room for packed point locations, or records of narrow rows with theirs, behind its workspace
(flexconv_workspace_bytes_best) against the same call in a workspace of the smallest size, which reads the tensors
themselves: the same bits, and both within the oracle's tolerance.  That the records were made, and where they lie, is read from
the workspace."""
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


def up256(n):
    return -(-n // 256) * 256


def expected_records(pos, rows):
    """numpy [B,3,N] and the gathered rows [B,W,N] -> the bytes behind the workspace: (x, y, z, 0) a point, or for W <= 16 four quads
    (component t of (x, y, z, 1), channels R t .. R t + 2) and, R = 4, behind all of them the channels 4 t + 3."""
    B, _, N = pos.shape
    at = torch.from_numpy(pos).transpose(1, 2)
    if rows.shape[1] > 16:
        return torch.cat([at, torch.zeros(B, N, 1)], 2).reshape(-1)
    R = -(-rows.shape[1] // 4)
    ch = torch.zeros(B, N, 4 * R)
    ch[:, :, :rows.shape[1]] = torch.from_numpy(rows).transpose(1, 2)
    ch = ch.reshape(B, N, 4, R)
    rec = torch.zeros(B, N, 4, 4)
    rec[..., 0] = torch.cat([at, torch.ones(B, N, 1)], 2)
    rec[..., 1:1 + min(R, 3)] = ch[..., :3]
    return torch.cat([rec.reshape(-1)] + ([ch[..., 3].reshape(-1)] if R == 4 else []))


def compare(B, N, K, Din, Dout, layout, backward, hub=False):
    say(f"packed: B={B} N={N} K={K} {Din}->{Dout} layout={layout} hub={hub}")
    pos, nbr, feat, theta, bias, g = random_problem(40 + N + K, B, N, K, Din, Dout)
    if hub:                                  # point 3 is listed by every centre: a list of N entries, empty ones elsewhere
        nbr[:, -1, :] = 3
    a = (to_layout(feat, layout), dev(pos), dev(nbr), dev(theta), dev(bias))
    gd = to_layout(g, layout)
    edges = fx.flex_inedges_build(a[2])
    results = []
    for kind in (ExactWorkspace, BestWorkspace):
        w = kind(fx.OP_CONV_BWD if backward else fx.OP_CONV_FWD, B, N, K, Din, Dout, layout)
        w.ws.fill_(0x5A)
        if backward:
            r = fx.flexconv_bwd(*a, gd, layout=layout, in_edges=edges, workspace=w.ws)
            r += fx.flexconv_bwd(*a, gd, layout=layout, in_edges=edges, need_params=False, workspace=w.ws)[:1]
        else:
            r = (fx.flexconv_fwd(*a, layout=layout, workspace=w.ws),)
        w.check()
        if kind is BestWorkspace:
            want = expected_records(pos, g if backward else feat)
            at = w.need - up256(4 * want.numel())
            assert at >= fx.workspace_bytes(fx.OP_CONV_BWD if backward else fx.OP_CONV_FWD, B, N, K, Din, Dout, layout)
            got = w.ws[at:at + 4 * want.numel()].view(torch.int32).cpu()
            assert torch.equal(got, want.view(torch.int32))
        results.append(r)
    for x, y in zip(*results):
        assert torch.equal(x, y)
    if backward:
        assert rel_err(from_layout(results[1][0], layout), oracle.flexconv_bwd(feat, pos, nbr, theta, bias, g)[0]) <= TOL
    else:
        assert rel_err(from_layout(results[1][0], layout), oracle.flexconv_fwd(feat, pos, nbr, theta, bias)) <= TOL


# clouds around a tile of 32 / 48 points and around a packing block of 2048, K around a batch of eight, several clouds;
# gathered widths of one lane group per row (64) and of half a one (32), in both directions
@pytest.mark.parametrize("layout", [fx.BNC, fx.BCN], ids=["bnc", "bcn"])
@pytest.mark.parametrize("B,N,K,Din,Dout", [
    (1, 1, 1, 64, 64), (2, 47, 8, 64, 64), (1, 49, 9, 64, 64), (3, 97, 16, 64, 64), (1, 2049, 5, 64, 64),
    (2, 33, 3, 64, 128), (1, 300, 8, 64, 32), (1, 300, 12, 32, 64), (2, 2047, 8, 32, 32), (150, 17, 8, 64, 64),
])
def test_packed_locations_change_no_bit(B, N, K, Din, Dout, layout):
    compare(B, N, K, Din, Dout, layout, False)
    if Dout <= 64:                           # (rows wider than 64 channels read the tensor either way)
        compare(B, N, K, Din, Dout, layout, True)


# the feature gradient: two to four channels a quad with every remainder, clouds around the sixteen points of a wave and many
# that share a workgroup of eight waves, result widths that fill, leave and barely enter a block of 64, K around a batch of eight
@pytest.mark.parametrize("layout", [fx.BNC, fx.BCN], ids=["bnc", "bcn"])
@pytest.mark.parametrize("B,N,K,W,other", [
    (1, 1, 1, 5, 4), (1, 15, 3, 6, 64), (2, 16, 8, 7, 32), (1, 17, 9, 8, 65), (3, 63, 8, 9, 68), (1, 65, 16, 10, 3),
    (1, 257, 17, 9, 64), (2, 130, 8, 11, 130), (1, 300, 8, 12, 64), (2, 97, 5, 13, 64), (1, 5000, 8, 16, 20),
    (67, 17, 8, 9, 64), (300, 1, 1, 16, 8), (41, 16, 4, 5, 70), (19, 33, 9, 13, 64),
])
def test_records_over_lists_change_no_bit(B, N, K, W, other, layout):
    compare(B, N, K, other, W, layout, True)


def test_records_of_a_hub_point_and_empty_lists():
    compare(1, 500, 4, 64, 13, fx.BNC, True, hub=True)
    compare(2, 90, 8, 9, 9, fx.BCN, True, hub=True)


# the forward pass takes records from 2^17 points on, point-major where K is large enough for the widths
@pytest.mark.parametrize("layout", [fx.BNC, fx.BCN], ids=["bnc", "bcn"])
@pytest.mark.parametrize("B,N,K,W,other", [(1, 131072, 12, 5, 4), (2, 65537, 9, 9, 64), (1, 131073, 8, 12, 65), (3, 43701, 8, 7, 70),
                                             (8193, 16, 9, 8, 65), (1009, 130, 8, 9, 64)])
def test_records_change_no_bit(B, N, K, W, other, layout):
    compare(B, N, K, W, other, layout, False)


def test_parameter_gradients_alone_pack_only_beside_copies():
    # point-major tensors of listed widths are read as they are, and the packing would be the call's only preparation
    B, N, K, Din, Dout = 1, 700, 8, 64, 64
    pos, nbr, feat, theta, bias, g = random_problem(5, B, N, K, Din, Dout)
    for layout, packs in ((fx.BNC, False), (fx.BCN, True)):
        a = (to_layout(feat, layout), dev(pos), dev(nbr), dev(theta), dev(bias), to_layout(g, layout))
        edges = fx.flex_inedges_build(a[2])
        w = BestWorkspace(fx.OP_CONV_BWD, B, N, K, Din, Dout, layout)
        least = fx.workspace_bytes(fx.OP_CONV_BWD, B, N, K, Din, Dout, layout)
        w.ws[least:] = 0x5A
        _, gt, gb = fx.flexconv_bwd(*a, layout=layout, in_edges=edges, need_feat=False, workspace=w.ws)
        w.check()
        assert bool((w.ws[least:] != 0x5A).any()) == packs
        assert rel_err(gt.cpu().numpy(), oracle.flexconv_bwd(feat, pos, nbr, theta, bias, g)[1]) <= TOL


@pytest.mark.parametrize("layout", [fx.BNC, fx.BCN], ids=["bnc", "bcn"])
def test_parameter_gradients_on_tiles_pack_nothing(layout, B=2, N=700, K=8, Din=128, Dout=64):
    """Their kernels read the location tensor, copies or not."""
    pos, nbr, feat, theta, bias, g = random_problem(5, B, N, K, Din, Dout)
    a = (to_layout(feat, layout), dev(pos), dev(nbr), dev(theta), dev(bias), to_layout(g, layout))
    w = BestWorkspace(fx.OP_CONV_BWD, B, N, K, Din, Dout, layout)
    least = fx.workspace_bytes(fx.OP_CONV_BWD, B, N, K, Din, Dout, layout)
    w.ws[least:] = 0x5A
    _, gt, gb = fx.flexconv_bwd(*a, layout=layout, in_edges=fx.flex_inedges_build(a[2]), need_feat=False, workspace=w.ws)
    w.check()
    assert bool((w.ws[least:] == 0x5A).all())
    assert rel_err(gt.cpu().numpy(), oracle.flexconv_bwd(feat, pos, nbr, theta, bias, g)[1]) <= TOL
