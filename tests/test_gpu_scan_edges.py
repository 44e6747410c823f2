"""The pair-grouped scan against the small-batch path, which shares no code with
it but the estimator's arithmetic: the same ids and the same estimates, bit for
bit (no tolerance), over list lengths at the edges of tiles, groups and items,
code widths, dimensions whose query rows end in half a group of chunks, both
query tiles, every ring depth, and batches around one and two query tiles.
"""
import pytest
import torch

from paper_2409_09913_amd import erq

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

DEV = torch.device("cuda:0")
LENGTHS = [0, 1, 31, 32, 33, 63, 64, 65, 96, 97, 127, 129, 255, 257, 300, 513, 1025, 1100]


def make(dp, bits, planes=1, metric="l2"):
    g = torch.Generator(device=DEV).manual_seed(dp * 10 + bits)
    nlist = len(LENGTHS)
    assign = torch.repeat_interleave(torch.arange(nlist, device=DEV, dtype=torch.int32),
                                     torch.tensor(LENGTHS, device=DEV))
    assign = assign[torch.randperm(len(assign), device=DEV, generator=g)].contiguous()
    cent = torch.randn((nlist, dp), device=DEV, generator=g)
    x = cent[assign.long()] + torch.randn((len(assign), dp), device=DEV, generator=g)
    P = torch.linalg.qr(torch.randn((dp, dp), device=DEV, generator=g))[0].contiguous()
    ix = erq.Index(dp, bits, nlist, P, metric=metric)
    ix.build(x, cent, assign)
    if planes == 2:
        ix.set_query_planes(2)
    return ix, x, g


@pytest.mark.parametrize("dp,bits,planes,metric", [(64, 1, 1, "l2"), (64, 4, 1, "l2"), (128, 2, 1, "ip"),
                                                   (192, 3, 1, "l2"), (320, 5, 2, "l2"), (768, 4, 1, "l2"),
                                                   (832, 6, 1, "ip"), (960, 7, 2, "l2"), (1536, 8, 2, "ip")])
def test_pipeline_equals_small_batch(dp, bits, planes, metric):
    print("scan edges", dp, bits, planes, metric, flush=True)
    ix, x, g = make(dp, bits, planes, metric)
    q = x[torch.randint(len(x), (70,), device=DEV, generator=g)] + 0.3 * torch.randn((70, dp), device=DEV, generator=g)
    for nprobe, kk in ((1, 10), (3, 10), (len(LENGTHS), 20), (len(LENGTHS), 100)):
        for nq in (1, 32, 33, 65, 70):
            ix.set_small_batch(128)
            want = ix.search(q[:nq].contiguous(), nprobe, kk)
            ix.set_small_batch(0)
            for nqt, pd in ((0, 0), (1, 1), (1, 2), (2, 3), (2, 1), (1, 6), (2, 4)):
                try:
                    ix.set_tune(nqt, pd)
                except erq.ErqError:                      # not a schedule of this width
                    continue
                got = ix.search(q[:nq].contiguous(), nprobe, kk)
                assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
            ix.set_tune(0, 0)


@pytest.mark.parametrize("nq,nprobe", [(1, 1), (1, 5), (2, 18), (17, 18), (40, 7)])
@pytest.mark.parametrize("kk", [1, 20, 64, 65, 128, 129, 300])
def test_small_batch_slices(nq, nprobe, kk):
    """Slices that pass every key, a threshold's or their exact top-kk, against the pipeline."""
    print("slices", nq, nprobe, kk, flush=True)
    ix, x, g = make(128, 4)
    q = x[torch.randint(len(x), (nq,), device=DEV, generator=g)] + 0.3 * torch.randn((nq, 128), device=DEV, generator=g)
    ix.set_small_batch(128)
    got = ix.search(q, nprobe, kk)
    ix.set_small_batch(0)
    want = ix.search(q, nprobe, kk)
    assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])


def test_workspace_that_is_not_16_byte_aligned():
    """The same results from a workspace at an odd multiple of 8 bytes."""
    ix, x, g = make(128, 4)
    q = x[torch.randint(len(x), (300,), device=DEV, generator=g)] + 0.3 * torch.randn((300, 128), device=DEV, generator=g)
    c = torch.randn((16_500, 128), device=DEV, generator=g)
    for nprobe, k in ((5, 10), (18, 100)):
        want = ix.search(q, nprobe, k)
        buf = torch.empty(ix.search_workspace_size(300, nprobe, k) + 8, dtype=torch.uint8, device=DEV)
        got = ix.search(q, nprobe, k, ws=buf[8:])
        assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
    want = erq.coarse_probe(q, c, 20)
    buf = torch.empty((256 << 20) + 8, dtype=torch.uint8, device=DEV)
    got = torch.empty_like(want)
    rc = erq.load().erq_coarse_probe(q.data_ptr(), 300, c.data_ptr(), 16_500, 128, 20, 0, got.data_ptr(), None,
                                     buf[8:].data_ptr(), 256 << 20, torch.cuda.current_stream().cuda_stream)
    assert rc == 0 and torch.equal(got, want)
