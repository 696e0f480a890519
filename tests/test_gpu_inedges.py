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


def test_kept_centres():
    rng = np.random.default_rng(2)
    nbr = rng.integers(0, 5000, size=(2, 8, 5000)).astype(np.int32)
    sel = np.sort(np.stack([rng.choice(5000, 1250, replace=False) for _ in range(2)])).astype(np.int32)
    check(nbr, sel)


# full runs of the deal step, and both sides of the number of buckets up to which it orders a run in LDS (3072 of 1024 points)
@pytest.mark.parametrize("N", [1_100_001, 3_145_728, 3_145_729])
def test_random_tensors_of_many_buckets(N):
    say(f"in-edges N={N} K=8")
    g = torch.Generator("cuda").manual_seed(N)
    nbr = torch.randint(0, N, (1, 8, N), device="cuda", dtype=torch.int32, generator=g)
    off, src = fx.flex_inedges_build(nbr)
    tgt, at = torch.sort(nbr[0].t().reshape(-1), stable=True)
    assert torch.equal(src, (at // 8).int())
    assert torch.equal(off, torch.searchsorted(tgt, torch.arange(N + 1, device="cuda", dtype=torch.int32)).int())
