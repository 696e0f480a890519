"""The 64-point tile kernels (forward pass and feature gradient of layers wider than 64 gathered channels, and of widths
without a kernel of their own), at the sizes where they can go wrong: clouds around a tile and around one point, rows that
end inside a lane's four channels or inside an input block, output blocks that reach past the width, list lengths around
a step of eight slots, hub points, several clouds, both layouts."""
import numpy as np
import pytest
import torch

import oracle
import paper_1803_07289_amd as fx
from gpu_util import TOL, ExactWorkspace, dev, to_layout, from_layout, say
from helpers import rel_err
from test_gpu_parity import random_problem

pytestmark = pytest.mark.gpu


def check(seed, B, N, K, Din, Dout, layout, hub=False):
    say(f"tile: B={B} N={N} K={K} {Din}->{Dout} layout={layout} hub={hub}")
    pos, nbr, feat, theta, bias, g = random_problem(seed, B, N, K, Din, Dout)
    if hub:                                  # point 3 is listed by every centre: a list of N entries, empty ones elsewhere
        nbr[:, -1, :] = 3
    a = (to_layout(feat, layout), dev(pos), dev(nbr), dev(theta), dev(bias))
    edges = fx.flex_inedges_build(a[2])
    out = fx.flexconv_fwd(*a, layout=layout)
    gf, _, _ = fx.flexconv_bwd(*a, to_layout(g, layout), layout=layout, in_edges=edges, need_params=False)
    torch.cuda.synchronize()
    assert rel_err(from_layout(out, layout), oracle.flexconv_fwd(feat, pos, nbr, theta, bias)) <= TOL
    rgf, _, _ = oracle.flexconv_bwd(feat, pos, nbr, theta, bias, g)
    assert rel_err(from_layout(gf, layout), rgf) <= TOL


@pytest.mark.parametrize("layout", [fx.BNC, fx.BCN], ids=["bnc", "bcn"])
@pytest.mark.parametrize("B,N,K,Din,Dout", [
    (1, 1, 1, 128, 128), (1, 63, 7, 128, 64), (1, 64, 8, 128, 128), (2, 65, 9, 128, 256), (1, 130, 16, 256, 128),
    (3, 200, 17, 70, 90),        # ragged input block, ragged output block
    (1, 97, 8, 66, 3),           # two channels in the second input block, a three-channel result
    (1, 150, 5, 3, 70),          # rows of fewer than four channels
    (2, 80, 8, 5, 7),            # one narrow block
    (1, 300, 8, 640, 384),       # ten input blocks (scales past the table), two output blocks
])
def test_sizes_around_the_tile_and_its_blocks(B, N, K, Din, Dout, layout):
    check(70 + N + K, B, N, K, Din, Dout, layout)


@pytest.mark.parametrize("layout", [fx.BNC, fx.BCN], ids=["bnc", "bcn"])
@pytest.mark.parametrize("B,N,K,Din,Dout", [
    (1, 130, 8, 192, 192), (2, 65, 9, 129, 20), (1, 200, 8, 40, 130), (1, 97, 5, 17, 129), (1, 64, 8, 191, 257),
    (1, 150, 16, 320, 200),
])
def test_blocks_of_widths_between_the_multiples_of_128(B, N, K, Din, Dout, layout):
    """As many input blocks as the rows have, where the parameter gradients' padded copies have more."""
    check(80 + N + K, B, N, K, Din, Dout, layout)


def test_hub_point_and_empty_lists():
    check(5, 1, 500, 4, 128, 128, fx.BNC, hub=True)
    check(6, 2, 90, 8, 100, 70, fx.BNC, hub=True)


@pytest.mark.parametrize("B,N,K,Din,Dout", [
    (1, 1, 1, 128, 128), (1, 63, 7, 128, 256), (2, 65, 9, 256, 128), (3, 130, 16, 130, 70),
    (1, 3001, 8, 1024, 128),     # sixteen input blocks, three tiles per workgroup
])
def test_parameter_gradients_of_wide_layers(B, N, K, Din, Dout, layout=fx.BNC):
    say(f"tile parameter gradients: B={B} N={N} K={K} {Din}->{Dout} layout={layout}")
    pos, nbr, feat, theta, bias, g = random_problem(40 + N, B, N, K, Din, Dout)
    lay = lambda a: to_layout(a, layout)
    edges = fx.flex_inedges_build(dev(nbr))
    _, gt, gb = fx.flexconv_bwd(lay(feat), dev(pos), dev(nbr), dev(theta), dev(bias), lay(g), layout=layout, in_edges=edges)
    rt, rb = np.zeros(theta.shape), np.zeros(bias.shape)
    for b in range(B):
        p, f, up = (a[b].astype(np.float64) for a in (pos, feat, g))
        rows = f.T[nbr[b]]                                                   # [K, N, Din]
        for d in range(3):
            rt[d] += ((p[d][nbr[b]] - p[d])[:, :, None] * rows).sum(axis=0).T @ up.T
        rb += rows.sum(axis=0).T @ up.T
    assert rel_err(gt.cpu().numpy(), rt) <= TOL and rel_err(gb.cpu().numpy(), rb) <= TOL


@pytest.mark.parametrize("B,N,K,Din,Dout", [
    (1, 2049, 8, 512, 512),      # one point in the last tile
    (1, 2111, 16, 512, 512),     # one short of whole tiles, two steps of slots
    (2, 1056, 5, 512, 640),      # the last tile ends at half its points
    (3, 700, 9, 640, 384),       # several clouds, a workgroup's tiles across them
])
def test_parameter_gradients_in_blocks_of_128_channels(B, N, K, Din, Dout):
    """Clouds of enough tiles for the wider blocks (tile_grad_plan)."""
    test_parameter_gradients_of_wide_layers(B, N, K, Din, Dout)


@pytest.mark.parametrize("layout", [fx.BNC, fx.BCN], ids=["bnc", "bcn"])
@pytest.mark.parametrize("B,N,K,Din,Dout", [
    (1, 65, 8, 3, 100), (2, 70, 9, 101, 2),            # rows of fewer than four channels: copied
    (1, 1, 1, 65, 65), (1, 130, 8, 66, 129), (1, 97, 5, 67, 130), (2, 64, 16, 128, 131),     # a lane's four channels across the rows' end
    (1, 64, 8, 64, 128), (1, 33, 8, 128, 64), (1, 150, 8, 1, 65),
    (1, 2500, 8, 515, 514),                            # blocks of 128 channels
])
def test_parameter_gradients_at_the_rows_own_widths(B, N, K, Din, Dout, layout):
    test_parameter_gradients_of_wide_layers(B, N, K, Din, Dout, layout)


# widths that are contracted in fp32: one side of at most 64 channels, the other of 65 to 128
FP32_WIDTHS = [(64, 128), (128, 64), (100, 50), (3, 100), (65, 64), (64, 65), (127, 2)]


def parameter_gradients(pos, nbr, feat, g):
    theta, bias = np.zeros((3, feat.shape[1], g.shape[1]), np.float32), np.zeros((feat.shape[1], g.shape[1]), np.float32)
    lay = lambda a: to_layout(a, fx.BNC)
    edges = fx.flex_inedges_build(dev(nbr))
    _, gt, gb = fx.flexconv_bwd(lay(feat), dev(pos), dev(nbr), dev(theta), dev(bias), lay(g), layout=fx.BNC, in_edges=edges, need_feat=False)
    return gt.cpu().numpy(), gb.cpu().numpy()


@pytest.mark.parametrize("Din,Dout", FP32_WIDTHS)
@pytest.mark.parametrize("N,at", [(1, 0), (300, 299), (20_000, 7777)])
def test_parameter_gradients_of_one_point_are_products_rounded_once(Din, Dout, N, at):
    say(f"tile parameter gradients of point {at} of {N}, {Din}->{Dout}")
    pos, nbr, feat, theta, bias, g = random_problem(13, 1, N, 1, Din, Dout)
    g[:, :, np.arange(N) != at] = 0
    gt, gb = parameter_gradients(pos, nbr, feat, g)
    n = nbr[0, 0, at]
    f, up = feat[0, :, n], g[0, :, at]
    assert np.array_equal(gb, f[:, None] * up[None])
    for d in range(3):
        assert np.array_equal(gt[d], ((pos[0, d, n] - pos[0, d, at]) * f)[:, None] * up[None])


# sides that end in every part of 16 channels of a block: contracting waves without a channel write nothing
@pytest.mark.parametrize("Din,Dout", [(3, 100), (16, 65), (17, 80), (48, 81), (49, 96), (64, 97), (65, 16), (80, 17), (81, 33), (112, 64), (128, 1)])
@pytest.mark.parametrize("N", [130, 9000])
def test_fp32_parameter_gradients_take_nothing_from_what_the_workspace_held(Din, Dout, N, K=5):
    say(f"tile parameter gradients in a used workspace, N={N} {Din}->{Dout}")
    pos, nbr, feat, theta, bias, g = random_problem(15, 1, N, K, Din, Dout)
    a = (to_layout(feat, fx.BNC), dev(pos), dev(nbr), dev(theta), dev(bias), to_layout(g, fx.BNC))
    ws = ExactWorkspace(fx.OP_CONV_BWD_BUILD, 1, N, K, Din, Dout, fx.BNC)
    ws.ws.fill_(0xFF)
    _, gt, gb = fx.flexconv_bwd(*a, layout=fx.BNC, need_feat=False, workspace=ws.ws)
    ws.check()
    p, f, up = (x[0].astype(np.float64) for x in (pos, feat, g))
    rows = f.T[nbr[0]]
    assert rel_err(gb.cpu().numpy(), rows.sum(axis=0).T @ up.T) <= TOL
    for d in range(3):
        assert rel_err(gt[d].cpu().numpy(), ((p[d][nbr[0]] - p[d])[:, :, None] * rows).sum(axis=0).T @ up.T) <= TOL


@pytest.mark.parametrize("Din,Dout", FP32_WIDTHS)
@pytest.mark.parametrize("where", ["gradient", "feature", "feature of the last point's neighbour"])
@pytest.mark.parametrize("N", [300, 9000])
def test_infinities_reach_the_parameter_gradients_as_such(Din, Dout, where, N, K=8):
    say(f"tile parameter gradients, an infinite {where} among {N}, {Din}->{Dout}")
    pos, nbr, feat, theta, bias, g = random_problem(14, 1, N, K, Din, Dout)
    g = np.abs(g) + np.float32(0.1)                    # one sign: what is infinite stays so in the sum
    if where == "gradient":
        g[0, 1, 17] = -np.inf
    else:
        nbr[nbr == 17] = 18
        if where != "feature":
            nbr[0, 3, N - 1] = 17
        else:
            nbr[0, 3, 40:60] = 17
        feat[0, 1, 17] = np.inf
    gt, gb = parameter_gradients(pos, nbr, feat, g)
    with np.errstate(invalid="ignore"):
        p, f, up = (a[0].astype(np.float64) for a in (pos, feat, g))
        rows = f.T[nbr[0]]
        ref = [np.einsum("nc,no->co", ((p[d][nbr[0]] - p[d])[:, :, None] * rows).sum(axis=0), up.T) for d in range(3)]
        ref.append(np.einsum("nc,no->co", rows.sum(axis=0), up.T))
    assert np.isinf(ref[3]).any() and not np.isnan(ref[3]).any()
    for got, want in zip([gt[0], gt[1], gt[2], gb], ref):
        odd = ~np.isfinite(want)
        assert np.array_equal(got[odd], want[odd].astype(np.float32), equal_nan=True)
        assert rel_err(got[~odd], want[~odd]) <= TOL


@pytest.mark.parametrize("B,N,K,Din,Dout", [
    (1, 8192, 4, 33, 64), (2, 4096, 4, 50, 47), (1, 8191, 4, 50, 47),         # 64 x 64 channels, both sides of the line
    (1, 1 << 17, 3, 5, 6), (2, 1 << 16, 3, 20, 13), (1, (1 << 17) - 1, 3, 20, 13), (1, 1 << 17, 3, 5, 64), (1, 1 << 17, 3, 3, 5),
])
def test_parameter_gradients_of_narrow_layers_on_tiles(B, N, K, Din, Dout):
    test_parameter_gradients_of_wide_layers(B, N, K, Din, Dout)


# (chunks of workgroups a block are the smaller of its tiles and its share of the 256 CUs)
@pytest.mark.parametrize("partials,N,Din,Dout", [
    (16, 16 * 64, 128, 128), (17, 16 * 64 + 1, 128, 128), (64, 64 * 64, 128, 128), (64, 8129, 128, 128),
    (128, 24_513, 128, 128),                               # blocks of 128 channels
    (127, 127 * 64, 64, 128), (128, 20_000, 64, 128),      # in fp32
    (128, 128 * 64, 50, 50), (129, 128 * 64 + 1, 50, 50), (256, 256 * 64 + 1, 50, 50),
])
def test_partials_of_every_reduction(partials, N, Din, Dout):
    """Up to 16 partials a block, up to 128 and more: a kernel each."""
    say(f"{partials} partials")
    test_parameter_gradients_of_wide_layers(1, N, 8, Din, Dout)


@pytest.mark.parametrize("N,Din,Dout", [
    (85 * 64 * 129 + 1, 129, 16),     # three blocks of 64 channels, 129 and 130 tiles a workgroup
    (128 * 64 * 129 + 1, 65, 16),     # two, in fp32
    (128 * 64 * 129 + 1, 65, 65),     # two of 128 channels
])
def test_parameter_gradients_of_more_tiles_than_a_chain_of_sums(N, Din, Dout):
    """A workgroup's totals are written after 64 tiles, added to after 128 and once more at the end."""
    say(f"tile parameter gradients, long chains: N={N} {Din}->{Dout}")
    gen = torch.Generator(device="cuda").manual_seed(N)
    rand = lambda *shape: torch.rand(shape, generator=gen, device="cuda")
    pos, feat, g = rand(1, 3, N), rand(1, N, Din) - 0.5, rand(1, N, Dout) - 0.5
    near = torch.randint(-40, 41, (N,), generator=gen, device="cuda") + torch.arange(N, device="cuda")
    nbr = near.clamp(0, N - 1).to(torch.int32).reshape(1, 1, N)
    theta, bias = torch.zeros(3, Din, Dout, device="cuda"), torch.zeros(Din, Dout, device="cuda")
    _, gt, gb = fx.flexconv_bwd(feat, pos, nbr, theta, bias, g, layout=fx.BNC, need_feat=False)
    ids, up = nbr[0, 0].long(), g[0].double()
    rows = feat[0].double()[ids]
    assert rel_err(gb.cpu().numpy(), (rows.t() @ up).cpu().numpy()) <= TOL
    for d in range(3):
        ref = (rows * (pos[0, d].double()[ids] - pos[0, d].double())[:, None]).t() @ up
        assert rel_err(gt[d].cpu().numpy(), ref.cpu().numpy()) <= TOL


@pytest.mark.parametrize("Din,Dout", [(64, 13), (64, 9), (128, 128), (70, 90), (64, 64)])
@pytest.mark.parametrize("bad", [np.nan, np.inf])
def test_unlisted_point_without_a_location_has_no_gradient(Din, Dout, bad):
    """A point that no centre lists gets a zero feature gradient also where its own location is no number."""
    B, N, K, at, to = 1, 150, 7, 20, 3
    say(f"tile: unlisted point at {bad}, {Din}->{Dout}")
    pos, nbr, feat, theta, bias, g = random_problem(90, B, N, K, Din, Dout)
    nbr[nbr == at] = at + 1
    nbr[:, :, at] = to                       # it lists point 3 only, whose gradient is no number then
    ref, _, _ = oracle.flexconv_bwd(feat, pos, nbr, theta, bias, g)
    pos[:, :, at] = bad
    edges = fx.flex_inedges_build(dev(nbr))
    gf, _, _ = fx.flexconv_bwd(to_layout(feat, fx.BNC), dev(pos), dev(nbr), dev(theta), dev(bias), to_layout(g, fx.BNC),
                               layout=fx.BNC, in_edges=edges, need_params=False)
    torch.cuda.synchronize()
    gf = from_layout(gf, fx.BNC)
    assert (np.asarray(gf)[:, :, at] == 0).all()
    rest = np.arange(N) != to
    assert rel_err(np.asarray(gf)[:, :, rest], ref[:, :, rest]) <= TOL
