"""More rows than one launch can give a wave each (2^26 rows are 2^32 threads):
17 GB of rows at 64 dimensions, far from the origin, so that the norms decide how
the distances round and a row whose norm is missing gets another list.
"""
import pytest
import torch

from paper_2409_09913_amd import erq

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

DEV = torch.device("cuda:0")
N, DP, C = (1 << 26) + 33, 64, 5


@pytest.fixture(scope="module")
def x():
    if torch.cuda.mem_get_info()[0] < 64 << 30:
        pytest.skip("needs 64 GB of device memory")
    yield torch.randn((N, DP), device=DEV, generator=torch.Generator(device=DEV).manual_seed(1)).add_(1000.0)
    torch.cuda.empty_cache()


def test_kmeans(x):
    cent, got = erq.kmeans(x, C, iters=1, seed=3)
    for lo in (0, (1 << 24) - 500, (1 << 25) - 500, N - 1000):
        want = erq.coarse_probe(x[lo:lo + 1000], cent, 1)[:, 0]
        assert int((got[lo:lo + 1000] != want).sum()) == 0, lo
    assert int(torch.bincount(got, minlength=C).sum()) == N


def test_quantize(x):
    got = erq.quantize(x, 3)
    for lo in (0, (1 << 24) - 500, (1 << 25) - 500, N - 1000):
        for a, b in zip(got, erq.quantize(x[lo:lo + 1000].contiguous(), 3)):
            assert int((a[lo:lo + 1000] != b).sum()) == 0, lo


def test_build_and_search(x):
    """A two-stage index: its results on both scan paths are those of an index of the returned rows alone."""
    y = x - 1000.0
    q = torch.randn((64, DP), device=DEV, generator=torch.Generator(device=DEV).manual_seed(2))
    P, cent = torch.eye(DP, device=DEV), y[::1 << 15].contiguous()
    ix = erq.Index(DP, 2, cent.shape[0], P)
    ix.set_two_stage(8.0)                             # no bound fails at 8
    ix.build(y, cent)
    ix.set_small_batch(0)
    ids, est = ix.search(q, 8, 10)
    ix.set_two_stage(0.0)
    ix.set_small_batch(128)
    ids1, est1 = ix.search(q, 8, 10)
    ix.close()
    assert int((ids != ids1).sum()) == 0 and int((est != est1).sum()) == 0
    rows = ids.unique()
    part = erq.Index(DP, 2, cent.shape[0], P)
    part.build(y[rows].contiguous(), cent)
    ids2, est2 = part.search(q, 8, 10)
    part.close()
    assert int((rows[ids2] != ids).sum()) == 0 and int((est2 != est).sum()) == 0


def test_probe_and_rerank(x):
    """2^24 queries and more: a workgroup of 256 threads each in the selection and the re-rank."""
    nq = (1 << 24) + 5
    q, cent = x[:nq], x[-3:].contiguous()
    probes, pd = erq.coarse_probe(q, cent, 2, with_dist=True)
    ix = erq.Index(DP, 1, 3, torch.eye(DP, device=DEV))
    ix.build(cent, cent, keep_raw=True)
    cand = torch.arange(nq, device=DEV).remainder(3)[:, None].repeat(1, 2)
    cand[:, 1] = 2
    ids, d = ix.rerank(q, cand, 1)
    for lo in (0, (1 << 22) - 500, (1 << 23) - 500, nq - 1000):
        at = slice(lo, lo + 1000)
        p1, d1 = erq.coarse_probe(q[at].contiguous(), cent, 2, with_dist=True)
        assert int((p1 != probes[at]).sum()) == 0 and int((d1 != pd[at]).sum()) == 0, lo
        i1, d1 = ix.rerank(q[at].contiguous(), cand[at].contiguous(), 1)
        assert int((i1 != ids[at]).sum()) == 0 and int((d1 != d[at]).sum()) == 0, lo
    ix.close()
