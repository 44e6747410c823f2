"""The fused nearest-centroid assignment (k-means, index build) against the
probe's distances and selection, at the edges of its tiles and of its split of
the columns: the same list for every row, ties to the lower list.
"""
import numpy as np
import pytest
import torch

from paper_2409_09913_amd import erq

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

DEV = torch.device("cuda:0")


def rows(n, dp, seed, dup=0):
    g = torch.Generator(device=DEV).manual_seed(seed)
    x = torch.randn((n, dp), device=DEV, generator=g)
    if dup:
        x[dup:2 * dup] = x[:dup]
    return x


@pytest.mark.parametrize("n,dp,C", [(1, 64, 1), (127, 64, 31), (128, 128, 32), (129, 64, 33), (300, 192, 127),
                                    (1000, 64, 128), (1000, 128, 129), (2001, 64, 1000), (4097, 320, 257),
                                    (200_000, 64, 130)])
def test_assignment_equals_probe(n, dp, C):
    print("assign", n, dp, C, flush=True)
    x = rows(n, dp, n + C, dup=C // 3)
    cent, got = erq.kmeans(x, C, iters=0, seed=C)
    want = erq.coarse_probe(x, cent, 1)[:, 0]
    assert torch.equal(got, want)


@pytest.mark.parametrize("metric", ["l2", "ip", "cosine"])
def test_build_lists_equal_probe(metric):
    n, dp, C = 3001, 128, 77
    x, cent = rows(n, dp, 5), rows(C, dp, 6)
    cent[40] = cent[7]                                # a tie for every row of list 7
    P = torch.eye(dp, device=DEV)
    ix = erq.Index(dp, 4, C, P, metric=metric)
    ix.build(x, cent)
    off, ids = (t.cpu().numpy() for t in ix.export()[:2])
    ix.close()
    y = x / torch.linalg.vector_norm(x, dim=1, keepdim=True) if metric == "cosine" else x
    d = erq.coarse_probe(y, cent, 1, metric=metric)[:, 0].cpu().numpy()
    got = np.empty(n, np.int64)
    got[ids] = np.repeat(np.arange(C), np.diff(off))
    differ = (got != d).mean()
    assert differ <= (0.01 if metric == "cosine" else 0.0)    # cosine: torch's unit rows differ in the last bit
    assert off[41] == off[40]


@pytest.mark.parametrize("n,dp,C", [(50, 64, 3), (5000, 64, 2), (3000, 1088, 7)])
def test_means_of_long_lists(n, dp, C):
    """Lists longer than one partial sum (1024 members): means of the members in FP64, rounded once."""
    x = rows(n, dp, 3)
    c0, a0 = erq.kmeans(x, C, iters=0, seed=1)
    c1, _ = erq.kmeans(x, C, iters=1, seed=1)
    for l in range(C):
        m = x[a0 == l].double()
        want = (m.mean(0) if len(m) else c0[l].double()).float()
        assert torch.allclose(c1[l], want, rtol=2 ** -23, atol=1e-12 + 2.0 ** -50 * float(m.abs().sum(0).max()) / max(len(m), 1))


def plant(kind, x, c):
    """Rows and centroids whose distances overflow or are not numbers, some of them or all."""
    inf, nan = float("inf"), float("nan")
    n, C = len(x), len(c)
    if kind == "all overflow":
        x *= 1e19
        c *= 1e19
    elif kind == "last centroids overflow":
        x *= 1e19
        c[C - 3:] *= 1e19
    elif kind == "first centroids overflow":
        x *= 1e19
        c[:3] *= 1e19
    elif kind == "some rows overflow":
        x[n // 2:] *= 1e19
        c *= 1e19
    elif kind == "nan":
        x[n // 3, 5] = nan
        c[C // 2, 7] = -nan
        c[C - 1, 3] = nan
    elif kind == "inf":
        x[n // 3, 5], x[n // 2, 9] = inf, -inf
        c[0, 5], c[C // 2, 7] = inf, -inf


@pytest.mark.parametrize("kind", ["all overflow", "last centroids overflow", "first centroids overflow",
                                  "some rows overflow", "nan", "inf"])
@pytest.mark.parametrize("metric", ["l2", "ip"])
@pytest.mark.parametrize("n,dp,C", [(300, 64, 100), (5000, 128, 700), (40_000, 64, 300)])
def test_lists_of_distances_that_are_not_numbers(n, dp, C, metric, kind):
    """The order is the probe's there, too."""
    print("assign", n, dp, C, metric, kind, flush=True)
    x, cent = rows(n, dp, 1), rows(C, dp, 2)
    plant(kind, x, cent)
    ix = erq.Index(dp, 4, C, torch.eye(dp, device=DEV), metric=metric)
    ix.build(x, cent)
    off, ids = ix.export()[:2]
    ix.close()
    got = torch.empty(n, dtype=torch.int64, device=DEV)
    got[ids] = torch.repeat_interleave(torch.arange(C, device=DEV), off.diff())
    want = erq.coarse_probe(x, cent, 1, metric=metric)[:, 0]
    assert int((got != want).sum()) == 0
