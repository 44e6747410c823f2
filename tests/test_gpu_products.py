"""The BF16 hi/lo products of the probe and the rotation at the edges of every
tile shape they choose (one row, one tile, few rows, 2 x 1 and 2 x 2 tiles per
wave, 256 x 128 tiles through LDS), against FP64.

Bound per value: each product is off by at most 2^-15 |a_i b_i| (split residuals
and the dropped lo.lo) and the FP32 sum of 3 K terms by its forward error bound;
a distance takes twice that and the rounding of its three terms.
"""
import numpy as np
import pytest
import torch

from paper_2409_09913_amd import erq

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

DEV = torch.device("cuda:0")
U = 2.0 ** -24


@pytest.mark.parametrize("n,nl,dp", [(1, 1, 64), (1, 33, 64), (31, 300, 128), (32, 129, 192), (33, 65, 64),
                                     (129, 700, 320), (700, 5000, 64), (1025, 4100, 128), (5000, 300, 64),
                                     (2049, 8200, 64), (4100, 2055, 128)])
@pytest.mark.parametrize("metric", ["l2", "ip"])
def test_probe_distances(n, nl, dp, metric):
    print("probe products", n, nl, dp, metric, flush=True)
    g = torch.Generator(device=DEV).manual_seed(n + nl)
    q = torch.randn((n, dp), device=DEV, generator=g)
    c = torch.randn((nl, dp), device=DEV, generator=g)
    k = min(nl, 1024)
    probes, d = erq.coarse_probe(q, c, k, with_dist=True, metric=metric)
    p = probes.long()
    ip = (q.double() @ c.double().T).gather(1, p)
    mag = (q.double().abs() @ c.double().abs().T).gather(1, p)
    err = (2.0 ** -15 + 3 * dp * U / (1 - 3 * dp * U)) * mag
    if metric == "l2":
        n2 = (q.double() ** 2).sum(1)[:, None] + (c.double() ** 2).sum(1)[p]
        want, tol = n2 - 2 * ip, 2 * err + (dp + 3) * U * (n2 + 2 * mag)
    else:
        want, tol = -ip, err
    assert bool(((d.double() - want).abs() <= tol).all())
    assert bool((d[:, 1:] >= d[:, :-1]).all())
    if k == nl:                                       # every column once
        assert torch.equal(p.sort(1).values, torch.arange(nl, device=DEV).expand(n, nl))


@pytest.mark.parametrize("n,dp", [(1, 64), (33, 128), (257, 192), (3000, 128), (9000, 960)])
def test_rotation(n, dp):
    g = torch.Generator(device=DEV).manual_seed(n)
    x = torch.randn((n, dp), device=DEV, generator=g)
    P = torch.linalg.qr(torch.randn((dp, dp), device=DEV, generator=g))[0].contiguous()
    got = erq.rotate(x, P, precision=2).double()
    want = x.double() @ P.double()
    mag = x.double().abs() @ P.double().abs()
    assert bool(((got - want).abs() <= (2.0 ** -15 + 3 * dp * U / (1 - 3 * dp * U)) * mag).all())


@pytest.mark.parametrize("dp", [64, 128, 320, 768, 1088])
def test_fp32_rotation_does_not_depend_on_the_batch(dp):
    """One chain of fused multiply-adds per output, whatever tile shape the batch gets."""
    g = torch.Generator(device=DEV).manual_seed(dp)
    x = torch.randn((14_000, dp), device=DEV, generator=g) * torch.exp(2 * torch.randn((14_000, 1), device=DEV, generator=g))
    P = torch.randn((dp, dp), device=DEV, generator=g)
    want = erq.rotate(x, P).view(torch.int32)
    for n in (1, 15, 17, 33, 500, 1400, 3001):
        got = erq.rotate(x[:n].contiguous(), P).view(torch.int32)
        assert torch.equal(got, want[:n]), n


@pytest.mark.parametrize("n,nl,dp", [(32, 32_769, 64), (64, 32_800, 64), (65, 32_769, 64), (128, 33_000, 192),
                                     (257, 16_500, 64), (300, 20_000, 128), (384, 16_400, 64), (200, 16_384, 1536),
                                     (255, 16_390, 1600), (900, 4_400, 1536)])
def test_probe_does_not_depend_on_the_batch(n, nl, dp):
    """Few queries over many lists (128 x 128 tiles among others) against the same queries 16 at a time."""
    print("probe products", n, nl, dp, flush=True)
    g = torch.Generator(device=DEV).manual_seed(n + nl)
    q = torch.randn((n, dp), device=DEV, generator=g)
    c = torch.randn((nl, dp), device=DEV, generator=g)
    probes, d = erq.coarse_probe(q, c, 100, with_dist=True)
    for lo in range(0, n, 16):
        p1, d1 = erq.coarse_probe(q[lo:lo + 16].contiguous(), c, 100, with_dist=True)
        assert torch.equal(p1, probes[lo:lo + 16]) and torch.equal(d1, d[lo:lo + 16]), lo


@pytest.mark.parametrize("n,dp", [(10_000, 64), (4100, 128), (1000, 768), (1025, 1024), (200, 4096), (700, 704)])
def test_rotation_in_turns(n, dp):
    """Scratch cut in parts (planes of the rows, of P or of both between 2 and 4 MiB) against a few rows at a time."""
    g = torch.Generator(device=DEV).manual_seed(n)
    x = torch.randn((n, dp), device=DEV, generator=g)
    P = torch.randn((dp, dp), device=DEV, generator=g)
    got = erq.rotate(x, P, precision=2)
    for lo in range(0, n, 61 if n <= 1025 else 499):
        assert torch.equal(got[lo:lo + 40], erq.rotate(x[lo:lo + 40].contiguous(), P, precision=2)), lo


def test_timer_names():
    """"rotate" counts rotations launched by themselves; a search's is part of the probe's launch."""
    g = torch.Generator(device=DEV).manual_seed(5)
    x = torch.randn((500, 128), device=DEV, generator=g)
    P = torch.linalg.qr(torch.randn((128, 128), device=DEV, generator=g))[0].contiguous()
    ix = erq.Index(128, 4, 8, P)
    calls = [(lambda: erq.rotate(x, P, precision=2), 1, 0), (lambda: erq.coarse_probe(x, x[:8].contiguous(), 3), 0, 1),
             (lambda: ix.build(x, x[:8].contiguous()), 1, 1), (lambda: ix.search(x, 4, 5), 0, 1)]
    erq.profile_enable(True)
    erq.profile_read("rotate", reset=True)
    try:
        for call, rotate, probe in calls:
            call()
            assert (erq.profile_read("rotate")[1], erq.profile_read("probe")[1]) == (rotate, probe)
            erq.profile_read("rotate", reset=True)
    finally:
        erq.profile_enable(False)
    ix.close()
