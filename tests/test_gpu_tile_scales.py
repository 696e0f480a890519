"""Wide gathers (more than one block of 64 input channels) where the blocks differ in scale: a block that is zero, groups of
channels far apart in magnitude, and the rounding of the sum over the blocks.  A block's share of the result may cost
bits only next to what it is added to, not next to what the point has in other blocks."""
import numpy as np
import pytest
import torch

import oracle
import paper_1803_07289_amd as fx
from gpu_util import TOL, dev, to_layout, from_layout, say
from test_gpu_dynamic_range import rel_err_per_channel
from test_gpu_parity import random_problem

pytestmark = pytest.mark.gpu


def forward_and_feature_gradient(pos, nbr, feat, theta, bias, g, layout=fx.BNC):
    a = (to_layout(feat, layout), dev(pos), dev(nbr), dev(theta), dev(bias))
    out = fx.flexconv_fwd(*a, layout=layout)
    gf, _, _ = fx.flexconv_bwd(*a, to_layout(g, layout), layout=layout, need_params=False)
    torch.cuda.synchronize()
    return from_layout(out, layout), from_layout(gf, layout)


def check(pos, nbr, feat, theta, bias, g, layout=fx.BNC):
    out, gf = forward_and_feature_gradient(pos, nbr, feat, theta, bias, g, layout)
    rgf, _, _ = oracle.flexconv_bwd(feat, pos, nbr, theta, bias, g)
    errs = (rel_err_per_channel(out, oracle.flexconv_fwd(feat, pos, nbr, theta, bias), 1), rel_err_per_channel(gf, rgf, 1))
    say(f"  per-channel rel err: fwd {errs[0]:.2e} grad_feat {errs[1]:.2e}")
    assert max(errs) <= TOL, errs


@pytest.mark.parametrize("magnitude", [1.0, 1e-6, 1e-12])
@pytest.mark.parametrize("zero", [0, 1, 2], ids=["first", "middle", "last"])
@pytest.mark.parametrize("width,other", [(128, 64), (192, 192), (256, 128), (384, 256)])
def test_a_block_of_zeros_costs_the_others_nothing(width, other, zero, magnitude):
    blocks = (width + 63) // 64
    at = {0: 0, 1: blocks // 2, 2: blocks - 1}[zero]
    say(f"zero block {at} of {blocks}, {width}<->{other}, magnitude {magnitude}")
    for Din, Dout in ((width, other), (other, width)):           # the forward pass, the feature gradient gather `width`
        pos, nbr, feat, theta, bias, g = random_problem(60 + width + zero, 1, 150, 8, Din, Dout)
        pos *= 0.02
        wide = feat if Din == width else g
        wide *= np.float32(magnitude)
        wide[:, 64 * at:64 * at + 64] = 0
        check(pos, nbr, feat, theta, bias, g)


@pytest.mark.parametrize("second", [1e-8, 1e-16, 1e8, 1e16])
@pytest.mark.parametrize("layout", [fx.BNC, fx.BCN], ids=["bnc", "bcn"])
def test_groups_of_channels_keep_their_own_scale(second, layout):
    """Two groups of 128 channels that do not meet (block-diagonal parameters), far apart in scale."""
    say(f"groups, second at {second} of the first, layout={layout}")
    C = 256
    pos, nbr, feat, theta, bias, g = random_problem(77, 1, 200, 8, C, C)
    theta[:, :128, 128:] = theta[:, 128:, :128] = bias[:128, 128:] = bias[128:, :128] = 0
    feat[:, 128:] *= np.float32(second)
    g[:, 128:] *= np.float32(second)
    check(pos, nbr, feat, theta, bias, g, layout)


@pytest.mark.parametrize("C", [64, 128, 512])
def test_error_does_not_grow_with_the_input_blocks(C):
    """2-norm error of ordinary data.  What every width has in common: eight fp32 sums per aggregate, 22-bit halves, and per
    block eight partial sums that the matrix op rounds down by up to 2^-23, here 1.45e-7 together.  The blocks' results
    are added to nearest, 2^-25 each at random: 1.57e-7 at eight.  The bound leaves a quarter; with all products of all
    blocks in one chain of the matrix op's sums it was 2.7e-7 at two blocks and 5.1e-7 at eight."""
    pos, nbr, feat, theta, bias, g = random_problem(5, 1, 400, 8, C, C)
    out, gf = forward_and_feature_gradient(pos, nbr, feat, theta, bias, g)
    ref = oracle.flexconv_fwd(feat, pos, nbr, theta, bias)
    rgf, _, _ = oracle.flexconv_bwd(feat, pos, nbr, theta, bias, g)
    errs = [float(np.linalg.norm(x - y) / np.linalg.norm(y)) for x, y in ((out, ref), (gf, rgf))]
    say(f"{C}->{C}: 2-norm rel err fwd {errs[0]:.2e} grad_feat {errs[1]:.2e}")
    assert max(errs) <= 2e-7, errs


@pytest.mark.parametrize("N,C,adds", [(500, 128, 2), (2000, 128, 2), (20_000, 128, 10), (40_000, 512, 128)])
def test_error_of_the_parameter_gradients(N, C, adds):
    """2-norm error of the sums over all points.  Terms carry three 8-bit pieces and 32 of them go through six sums of the
    matrix op, which rounds down, with the sign of every second 32 turned round: with the aggregates' own rounding 1.0e-7,
    taken as 1.2e-7.  The results are added to nearest: rms at most 2^-24 / sqrt(3) of the running total, whose square
    grows with the additions, `adds` of them per total.  (Measured 1.0e-7, 1.0e-7, 1.1e-7, 2.2e-7; with chains of eight
    steps of one sign 2.6e-7 and 3.2e-7 in the last two.)"""
    bound = (1.2e-7 ** 2 + 2.0 ** -48 / 3 * adds / 2) ** 0.5
    rng = np.random.default_rng(N + C)
    pos = torch.from_numpy(rng.random((1, 3, N), dtype=np.float32)).cuda()
    nbr = torch.from_numpy(((np.arange(N)[None, None] + rng.integers(-20, 21, size=(1, 8, N))) % N).astype(np.int32)).cuda()
    feat, g = (torch.from_numpy(rng.standard_normal((1, N, C), dtype=np.float32)).cuda() for _ in range(2))
    theta, bias = torch.zeros((3, C, C), device="cuda"), torch.zeros((C, C), device="cuda")
    _, gt, gb = fx.flexconv_bwd(feat, pos, nbr, theta, bias, g, layout=fx.BNC, need_feat=False)
    got = torch.cat([gt, gb[None]]).double().cpu().numpy()
    p, n, f, up = pos[0].double().cpu(), nbr[0].long().cpu(), feat[0].double().cpu(), g[0].double().cpu()
    agg = torch.zeros((4, N, C), dtype=torch.float64)
    for k in range(8):
        rows, dp = f[n[k]], p[:, n[k]] - p
        for d in range(3):
            agg[d] += dp[d][:, None] * rows
        agg[3] += rows
    ref = np.stack([(a.t() @ up).numpy() for a in agg])
    err = float(np.linalg.norm(got - ref) / np.linalg.norm(ref))
    say(f"{N} points {C}->{C}: 2-norm rel err of the parameter gradients {err:.2e}")
    assert err <= bound, (err, bound)


def test_replays_of_a_captured_wide_layer():
    """Forward and all gradients of a layer whose parameter gradients' totals move to the partials in memory (more than 64
    tiles per workgroup), in a graph: every replay gives the eager call's bits, with eager work in between."""
    N, C = 20_000, 512
    rng = np.random.default_rng(3)
    pos = dev(rng.random((1, 3, N), dtype=np.float32))
    nbr = dev(((np.arange(N)[None, None] + rng.integers(-20, 21, size=(1, 8, N))) % N).astype(np.int32))
    feat, g = (dev(rng.standard_normal((1, N, C), dtype=np.float32)) for _ in range(2))
    theta, bias = dev(rng.standard_normal((3, C, C), dtype=np.float32)), dev(rng.standard_normal((C, C), dtype=np.float32))
    edges = fx.flex_inedges_build(nbr)
    ws = [torch.empty(fx.workspace_bytes(op, 1, N, 8, C, C, fx.BNC), dtype=torch.uint8, device="cuda")
          for op in (fx.OP_CONV_FWD, fx.OP_CONV_BWD)]

    def step():
        return (fx.flexconv_fwd(feat, pos, nbr, theta, bias, layout=fx.BNC, workspace=ws[0]),
                *fx.flexconv_bwd(feat, pos, nbr, theta, bias, g, layout=fx.BNC, in_edges=edges, workspace=ws[1]))

    want = [t.clone() for t in step()]
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        outs = step()
    for r in range(3):
        say(f"replay {r}")
        for t in (*outs, *ws):
            t.fill_(7)
        graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(outs, want))
        assert all(torch.equal(a, b) for a, b in zip(step(), want))
