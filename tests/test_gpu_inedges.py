"""In-edge lists against a plain numpy transposition: around the bucket sizes of the bucketed build, list lengths past a
bucket's LDS (a hub point, lists sorted in global memory), repeats, every K class, kept-centre lists."""
import numpy as np
import pytest
import torch

import paper_1803_07289_amd as fx
from gpu_util import dev, say

pytestmark = pytest.mark.gpu


def lists(nbr, sel=None):
    B, K, N = nbr.shape
    tgt, src = [], []
    for b in range(B):
        cols = np.arange(N) if sel is None else sel[b]
        t = nbr[b][:, cols] + b * N
        tgt.append(t.ravel())
        src.append(np.broadcast_to(np.arange(len(cols)), t.shape).ravel())
    tgt, src = np.concatenate(tgt), np.concatenate(src)
    o = np.lexsort((src, tgt))
    return np.searchsorted(tgt[o], np.arange(B * N + 1)).astype(np.int32), src[o].astype(np.int32)


def check(nbr, sel=None):
    off, src = fx.flex_inedges_build(dev(nbr)) if sel is None else fx.flex_inedges_build_sub(dev(nbr), dev(sel))
    torch.cuda.synchronize()
    roff, rsrc = lists(nbr, sel)
    assert np.array_equal(off.cpu().numpy(), roff) and np.array_equal(src.cpu().numpy(), rsrc)


@pytest.mark.parametrize("B,N,K", [(1, 1, 1), (1, 1023, 8), (2, 1025, 8), (1, 4096, 3), (3, 511, 16), (1, 300, 100),
                                   (1, 40_000, 9)])
@pytest.mark.parametrize("local", [False, True])
def test_random_tensors(B, N, K, local):
    say(f"in-edges B={B} N={N} K={K} local={local}")
    rng = np.random.default_rng(N + K)
    if local:                                # neighbours near the centre: most of a wave's edges share a bucket
        nbr = (np.arange(N)[None, None] + rng.integers(-20, 21, size=(B, K, N))) % N
    else:
        nbr = rng.integers(0, N, size=(B, K, N))
    check(nbr.astype(np.int32))


def test_hub_points_past_a_buckets_lds():
    rng = np.random.default_rng(1)
    nbr = rng.integers(0, 30_000, size=(1, 4, 30_000)).astype(np.int32)
    nbr[:, 1] = 7                            # 30 000 entries in one list
    nbr[:, 2] = np.where(np.arange(30_000) < 200, 9, nbr[:, 2])     # 200 + in another
    check(nbr)


# lists on both sides of what a thread (8, 16, 24 or 32, by K), a wave (64) and a workgroup order in a bucket's LDS, half of them with
# every centre twice
@pytest.mark.parametrize("K", [4, 8, 10, 11, 16, 17])
def test_lists_of_every_length(K):
    say(f"in-edges, lists of every length, K={K}")
    N, sizes = 20_000, [1, 2, 7, 8, 9, 15, 16, 17, 23, 24, 25, 31, 32, 33, 63, 64, 65, 66, 127, 128, 129, 1000, 2049]
    rng = np.random.default_rng(K)
    nbr = rng.integers(len(sizes), N, size=(1, K, N))
    for i, n in enumerate(sizes):
        own = rng.permutation(N)[:n] if i % 2 else np.repeat(rng.permutation(N)[: (n + 1) // 2], 2)[:n]
        for l in own:                        # a slot of this centre that no other list has taken
            nbr[0, np.argmax(nbr[0, :, l] >= len(sizes)), l] = i
    check(nbr.astype(np.int32))


@pytest.mark.parametrize("over", [-1, 0, 1])
def test_bucket_that_is_exactly_full(over):
    """As many edges as a bucket orders in LDS (12288), one fewer and one more, and no edge for its last targets."""
    say(f"in-edges, 12288 {over:+d} edges in a bucket")
    N, K, targets, full = 4096, 8, 1024, 12288 + over
    rng = np.random.default_rng(12)
    to = rng.integers(targets, N, size=K * N)
    to[rng.permutation(K * N)[:full]] = rng.integers(0, targets - 100, size=full)
    check(to.reshape(1, K, N).astype(np.int32))


# the one-launch build of small clouds: both sides of its lines (24576 edges a cloud, 2048 workgroups), stretches of one target and of
# many, lists past what a workgroup orders in LDS, kept centres of which some name no point
@pytest.mark.parametrize("B,N,K", [(1, 4096, 8), (1, 4097, 8), (1, 3072, 8), (1, 3073, 8), (3, 257, 9), (1, 2100, 1), (1, 180, 170), (2, 2600, 7), (2048, 16, 3), (2049, 16, 3), (1, 2, 2)])
def test_small_clouds(B, N, K):
    say(f"in-edges of small clouds B={B} N={N} K={K}")
    rng = np.random.default_rng(B + N)
    nbr = rng.integers(0, N, size=(B, K, N)).astype(np.int32)
    nbr[:, -1] = N // 2                                          # a hub in every cloud
    check(nbr)
    sel = rng.integers(-1, N + 1, size=(B, (N + 3) // 4)).astype(np.int32)
    got = fx.flex_inedges_build_sub(dev(nbr), dev(sel))
    torch.cuda.synchronize()
    for a, b in zip(got, lists(nbr, np.clip(sel, 0, N - 1))):
        assert np.array_equal(a.cpu().numpy(), b)


def test_hub_point_of_a_small_cloud():
    rng = np.random.default_rng(3)
    nbr = rng.integers(0, 4000, size=(2, 8, 4000)).astype(np.int32)
    nbr[1, 2:5] = 11                                             # 12 000 entries in one list
    nbr[1, 5, :300] = 12
    check(nbr)


def test_kept_centres():
    rng = np.random.default_rng(2)
    nbr = rng.integers(0, 5000, size=(2, 8, 5000)).astype(np.int32)
    sel = np.sort(np.stack([rng.choice(5000, 1250, replace=False) for _ in range(2)])).astype(np.int32)
    check(nbr, sel)


@pytest.mark.parametrize("Ns", [15_000, 15_001])             # both sides of three entries a list
def test_kept_centres_of_several_buckets(Ns):
    rng = np.random.default_rng(Ns)
    nbr = rng.integers(0, 40_000, size=(1, 8, 40_000)).astype(np.int32)
    nbr[0, 0, :40], nbr[0, 1, ::7] = 5, 6
    check(nbr, rng.permutation(40_000)[None, :Ns].astype(np.int32))


# the one-launch build over kept centres: more than a workgroup a CU, and both sides of its lines (768 workgroups, 2^22 edges walked)
@pytest.mark.parametrize("B,N,Ns,K", [(8, 9313, 2328, 9), (30, 1079, 269, 32), (30, 1079, 539, 32), (260, 40, 9, 5), (768, 50, 49, 3), (769, 50, 49, 3), (300, 300, 1, 2)])
def test_kept_centres_of_many_small_clouds(B, N, Ns, K):
    rng = np.random.default_rng(B + N)
    nbr = rng.integers(0, N, size=(B, K, N)).astype(np.int32)
    nbr[B // 2, 0] = N - 1
    check(nbr, np.stack([rng.permutation(N)[:Ns] for _ in range(B)]).astype(np.int32))


def check_large(nbr, sel=None):
    """The same on the device: the edges in (cloud, centre, slot) order, sorted by target without disturbing it."""
    B, K, N = nbr.shape
    off, src = fx.flex_inedges_build(nbr) if sel is None else fx.flex_inedges_build_sub(nbr, sel)
    cols = nbr if sel is None else nbr.gather(2, sel.long()[:, None, :].expand(-1, K, -1))
    tgt = (cols + N * torch.arange(B, device="cuda", dtype=torch.int32)[:, None, None]).transpose(1, 2).reshape(-1)
    tgt, at = torch.sort(tgt, stable=True)
    assert torch.equal(src, (at // K % cols.shape[2]).int())
    assert torch.equal(off, torch.searchsorted(tgt, torch.arange(B * N + 1, device="cuda", dtype=torch.int32)).int())


# full runs of the deal step, and both sides of the number of buckets up to which it orders a run in LDS (3072 of 1024 points); runs
# that cross clouds and slots, buckets of other sizes (512, 2048 points)
@pytest.mark.parametrize("B,N,K", [(1, 1_100_001, 8), (1, 3_145_728, 8), (1, 3_145_729, 8), (3, 250_001, 9), (2, 200_003, 16), (7, 300_001, 3)])
def test_random_tensors_of_many_buckets(B, N, K):
    say(f"in-edges B={B} N={N} K={K}")
    g = torch.Generator("cuda").manual_seed(N)
    check_large(torch.randint(0, N, (B, K, N), device="cuda", dtype=torch.int32, generator=g))


# runs that are ordered in LDS beside runs that are stored as they come, and one that a hub point's entries fill
@pytest.mark.parametrize("hub", [False, True])
def test_runs_with_and_without_locality(hub):
    N, K = 900_001, 8
    say(f"in-edges, half of the runs local, hub={hub}")
    g = torch.Generator("cuda").manual_seed(3)
    nbr = torch.randint(0, N, (1, K, N), device="cuda", dtype=torch.int32, generator=g)
    near = (torch.arange(N, device="cuda")[None] + torch.randint(-20, 21, (K // 2, N), device="cuda", generator=g)).clamp_(0, N - 1)
    nbr[0, ::2] = near.int()
    if hub:
        nbr[0, 3, 400_000:425_000] = 7       # 25 000 entries in one list
    check_large(nbr)


def test_many_kept_centres():
    # B * K * Ns edges enough for full runs; entries of a selection in no order
    B, N, K, Ns = 2, 500_001, 8, 330_001
    say(f"in-edges over kept centres B={B} N={N} Ns={Ns}")
    g = torch.Generator("cuda").manual_seed(4)
    nbr = torch.randint(0, N, (B, K, N), device="cuda", dtype=torch.int32, generator=g)
    sel = torch.stack([torch.randperm(N, device="cuda", generator=g)[:Ns] for _ in range(B)]).int()
    check_large(nbr, sel)
