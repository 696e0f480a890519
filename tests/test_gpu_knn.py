"""GPU parity for the grid k-nearest-neighbour search: the index tensor must equal the exhaustive CPU search bit for
bit (float32 squared distances, ties to the lower index) on generic, degenerate and tie-heavy clouds."""
import numpy as np
import pytest
import torch

import oracle
import paper_1803_07289_amd as fx
from gpu_util import ExactWorkspace, dev, say
from workloads import CONFIGS, make_inputs

pytestmark = pytest.mark.gpu


def _check(pos, K):
    nbr = fx.flex_knn(dev(pos), K)
    torch.cuda.synchronize()
    ref = oracle.knn(pos, K)
    got = nbr.cpu().numpy()
    bad = np.argwhere(got != ref)
    assert bad.size == 0, (bad[:5], got[tuple(bad[0])], ref[tuple(bad[0])])


@pytest.mark.parametrize("B,N,K", [(2, 3000, 8), (1, 5000, 16), (3, 700, 9), (1, 10, 10), (1, 1, 1), (2, 257, 1),
                                   (1, 2000, 32), (1, 1500, 5)])
def test_knn_uniform_cube(B, N, K):
    say(f"knn cube B={B} N={N} K={K}")
    pos = np.random.default_rng(N + K).random((B, 3, N)).astype(np.float32)
    _check(pos, K)


def test_knn_lattice_with_many_ties():
    rng = np.random.default_rng(1)
    pos = rng.integers(0, 12, size=(2, 3, 4000)).astype(np.float32)     # equal distances and coincident points
    _check(pos, 8)
    _check(pos * np.float32(0.37), 16)


def test_knn_degenerate_shapes():
    rng = np.random.default_rng(2)
    N = 3000
    flat = rng.random((1, 3, N)).astype(np.float32); flat[0, 2] = 0.25           # a plane
    line = np.zeros((1, 3, N), np.float32); line[0, 0] = rng.random(N)            # a line
    same = np.full((1, 3, 500), 1.5, np.float32)                                 # one location
    far = rng.random((1, 3, N)).astype(np.float32) * 0.5 + np.float32(1000.0)    # far from the origin: coarse float grid
    clumps = (rng.integers(0, 3, size=(1, 3, N)) * 100.0 + rng.normal(0, 0.01, (1, 3, N))).astype(np.float32)
    for name, pos, K in (("plane", flat, 8), ("line", line, 8), ("one location", same, 8), ("offset", far, 8),
                         ("clumps", clumps, 16)):
        say("knn", name)
        _check(pos, K)


# all against all up to 4096 points a cloud and 25 * 2^20 pairs; then the grid with 16, 8 and 4 lanes to a point and a thread each
@pytest.mark.parametrize("B,N,K", [(1, 4096, 12), (1, 4097, 12), (2, 3620, 4), (2, 3622, 4), (1, 12, 12), (5, 17, 16), (1, 4500, 1),
                                   (8, 4300, 9), (8, 4097, 2), (12, 5500, 4), (24, 5500, 8)])
def test_knn_on_both_sides_of_every_line(B, N, K):
    say(f"knn lanes B={B} N={N} K={K}")
    rng = np.random.default_rng(N + K)
    pos = rng.random((B, 3, N)).astype(np.float32)
    pos[B // 2] = rng.integers(0, 9, size=(3, N))                                # ties and coincident points
    pos[B - 1, 2] *= 0.01                                                        # a slab: empty cells around, many shells
    pos[B - 1, :, : N // 3] *= 0.05
    _check(pos, K)


def _check_fused(pos, K):
    """Lists are the oracle's, whose distances round every product and sum, or those under fma(dz, dz, fma(dx, dx, dy * dy))."""
    got, ref = fx.flex_knn(dev(pos), K).cpu().numpy(), oracle.knn(pos, K)
    others = np.argwhere((got != ref).any(axis=1))
    assert len(others) <= 1e-5 * got.size
    for b, l in others:
        d = pos[b] - pos[b, :, l : l + 1]
        yy, (x, _, z) = (d[1] * d[1]).astype(np.longdouble), d.astype(np.longdouble)        # 64 bits hold a product of two and nearly all sums
        d2 = (z * z + (x * x + yy).astype(np.float32).astype(np.longdouble)).astype(np.float32)
        assert np.array_equal(got[b, :, l], np.lexsort((np.arange(pos.shape[2]), d2))[:K]), (b, l)


# all against all, 16, 8 and 4 lanes to a point, a thread each: so many lists that some distances differ in their last bit alone
@pytest.mark.parametrize("B,N", [(12, 1400), (6, 5000), (9, 5461), (16, 6000), (24, 5500)])
def test_knn_ranks_by_the_fused_distance(B, N, K=32):
    say(f"knn rounding B={B} N={N}")
    _check_fused(np.random.default_rng(N).random((B, 3, N)).astype(np.float32), K)


# clouds searched a thread to a point although there are lanes to spare, and others of the same batch that are not: one layer of cells beyond
# 229376 entries and 16384 points, filled boxes beyond 3 * 2^19 entries
@pytest.mark.parametrize("B,N,K", [(2, 14_336, 8), (2, 14_337, 8), (4, 4097, 12), (4, 4097, 16), (3, 12_000, 8), (7, 9500, 4), (9, 5462, 32), (9, 5461, 32), (6, 11_000, 24)])
def test_knn_of_clouds_with_few_records_around(B, N, K):
    say(f"knn few records B={B} N={N} K={K}")
    rng = np.random.default_rng(N + K)
    pos = rng.random((B, 3, N)).astype(np.float32)
    pos[1::3, 2] = 0.25                                                          # a plane
    pos[2::3, 0] = (rng.random(pos[2::3, 0].shape) < 0.5) + 0.001 * pos[2::3, 0]       # two walls far apart
    _check_fused(pos, K)


def test_knn_degenerate_shapes_on_the_grid():
    rng = np.random.default_rng(2)
    N = 4500
    flat = rng.random((1, 3, N)).astype(np.float32); flat[0, 2] = 0.25
    line = np.zeros((1, 3, N), np.float32); line[0, 0] = rng.random(N)
    far = rng.random((1, 3, N)).astype(np.float32) * 0.5 + np.float32(1000.0)
    clumps = (rng.integers(0, 3, size=(1, 3, N)) * 100.0 + rng.normal(0, 0.01, (1, 3, N))).astype(np.float32)
    for name, pos, K in (("plane", flat, 8), ("line", line, 8), ("one location", np.full((1, 3, N), 1.5, np.float32), 8), ("offset", far, 8),
                         ("clumps", clumps, 32)):
        say("knn on the grid", name)
        _check(pos, K)


# the deal with 2 and 4 points a thread, 512 to 4096 cells a bucket, sparse and dense ones
@pytest.mark.parametrize("B,N,K", [(2, 131_000, 4), (1, 600_000, 4), (1, 1_100_000, 1)])
def test_knn_of_clouds_dealt_into_buckets(B, N, K):
    say(f"knn buckets B={B} N={N} K={K}")
    rng = np.random.default_rng(N)
    pos = rng.random((B, 3, N)).astype(np.float32)
    pos[:, :, : N // 3] *= np.float32(0.5)
    nbr = fx.flex_knn(dev(pos), K).cpu().numpy()
    assert np.array_equal(np.sort(nbr[:, 0]), np.broadcast_to(np.arange(N, dtype=np.int32), (B, N)))     # no two points coincide
    for l in rng.integers(0, N, size=48):
        for b in range(B):
            d = pos[b] - pos[b, :, l : l + 1]
            d2 = (d[0] * d[0] + d[1] * d[1]) + d[2] * d[2]
            assert np.array_equal(nbr[b, :, l], np.lexsort((np.arange(N), d2))[:K]), (b, l)


# most points in a few cells of a box that others stretch: a bucket of as many points as a workgroup sorts alone (8208) and one more, several
# such buckets that begin and end anywhere, a cloud without beside one with
@pytest.mark.parametrize("sizes", [(8208,), (8209,), (8192, 8209), (20_000, 9000, 100, 8300)])
@pytest.mark.parametrize("K", [8, 3])
def test_knn_of_clouds_that_stray_points_stretch(sizes, K):
    say(f"knn piles {sizes} K={K}")
    rng = np.random.default_rng(sum(sizes) + K)
    at = rng.permutation(27)[: len(sizes)]                                       # corners of a lattice, buckets apart
    p = [rng.random((3, n)) * 0.02 + 10.0 * np.array([[c // 9], [c // 3 % 3], [c % 3]]) for n, c in zip(sizes, at)]
    p.append(rng.random((3, 500)) * 25 + 1)
    p = np.concatenate(p, axis=1).astype(np.float32)
    p[:, 7], p[:, 8:12] = p[:, 5], p[:, 6:7]                                     # coincident points
    pos = np.stack([p[:, rng.permutation(p.shape[1])], rng.random(p.shape).astype(np.float32)])
    _check_fused(pos, K)
    for left in (0x7F, 0xFF):
        ws = ExactWorkspace(fx.OP_KNN, *pos.shape[::2], K, 1, 1, fx.BCN)
        ws.ws.fill_(left)
        got = fx.flex_knn(dev(pos), K, workspace=ws.ws)
        ws.check()
        assert torch.equal(got, fx.flex_knn(dev(pos), K))


# a lane group and a thread to a point
@pytest.mark.parametrize("N", [9000, 140_000])
@pytest.mark.parametrize("left", [0, 0x7F, 0xFF])
def test_knn_takes_nothing_from_what_the_workspace_held(N, left, K=8):
    say(f"knn N={N} in a workspace of {left:#x}")
    pos = np.random.default_rng(N).random((1, 3, N)).astype(np.float32)
    pos[0, :, : N // 2] *= np.float32(0.2)
    ws = ExactWorkspace(fx.OP_KNN, 1, N, K, 1, 1, fx.BCN)
    ws.ws.fill_(left)
    got = fx.flex_knn(dev(pos), K, workspace=ws.ws)
    ws.check()
    assert fx.flex_validate_neighbors(got) == 0
    assert torch.equal(got, fx.flex_knn(dev(pos), K))
    if N < 10_000:
        assert np.array_equal(got.cpu().numpy(), oracle.knn(pos, K))


@pytest.mark.parametrize("N", [600, 4500, 11_000])
def test_knn_infinite_locations(N):
    """At infinity a point is as far as can be from the others and no distance from its like."""
    pos = np.random.default_rng(8).random((1, 3, N)).astype(np.float32)
    pos[0, 0, 7], pos[0, 1, 9] = np.inf, -np.inf
    ref = oracle.knn(np.ascontiguousarray(np.delete(pos, [7, 9], axis=2)), 8)
    got = fx.flex_knn(dev(pos), 8).cpu().numpy()
    keep = np.delete(np.arange(N, dtype=np.int32), [7, 9])
    assert np.array_equal(got[:, :, keep], keep[ref])


@pytest.mark.parametrize("bits", [0x7fc00000, 0xffc00000])
def test_knn_location_that_is_no_number(bits, N=600):
    """A point without a location is nobody's neighbour, whichever sign its NaN has: the other points' lists are those
    of the cloud without it."""
    K, lost = 8, 77
    pos = np.random.default_rng(5).random((1, 3, N)).astype(np.float32)
    keep = np.delete(np.arange(N, dtype=np.int32), lost)
    ref = keep[oracle.knn(np.ascontiguousarray(pos[:, :, keep]), K)]
    pos[0, 1, lost] = np.array(bits, np.uint32).view(np.float32)
    got = fx.flex_knn(dev(pos), K).cpu().numpy()[:, :, keep]
    assert np.array_equal(got, ref)


@pytest.mark.parametrize("bits", [0x7fc00000, 0xffc00000])
def test_knn_location_that_is_no_number_on_the_grid(bits):
    test_knn_location_that_is_no_number(bits, N=4500)


def test_knn_room_cloud_matches_and_feeds_the_layers():
    """Room surfaces (the workload's geometry), 30k points: equal to the exhaustive search, and the tensor is a valid
    input of the other entry points."""
    x = make_inputs(CONFIGS[2], with_grad=False, n_override=30_000)
    _check(x.pos, 8)
    nbr = fx.flex_knn(dev(x.pos), 8)
    assert fx.flex_validate_neighbors(nbr) == 0
    assert torch.equal(nbr[0, 0].cpu(), torch.arange(30_000, dtype=torch.int32))   # jittered points: no coincidences
