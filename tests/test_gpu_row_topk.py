"""The probe's selection of the nearest centroids at the edges of its two routes
(a bound from chunk minima, the radix select): rows shorter and longer than a
turn of threads, k around its limits, ties (by column), and rows whose smallest
values crowd one chunk.  The distances come from the probe itself with k = all
columns or from integers, so the expected order is exact (no tolerance)."""
import pytest
import torch

from paper_2409_09913_amd import erq

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

DEV = torch.device("cuda:0")


@pytest.mark.parametrize("N", [1, 2, 63, 255, 256, 257, 1023, 1024, 1025, 1100, 2049, 4095, 4096, 4097, 8192, 9000])
@pytest.mark.parametrize("kind", ["spread", "ties", "crowded", "equal"])
def test_probe_order(N, kind):
    """Small integer vectors: every distance is a whole number below 2^24, exact in FP32."""
    print("row topk", N, kind, flush=True)
    g = torch.Generator(device=DEV).manual_seed(N)
    dp = 64
    q = torch.randint(-4, 5, (5, dp), device=DEV, generator=g).float()
    hi = {"spread": 15, "ties": 2, "crowded": 15, "equal": 1}[kind]
    c = torch.randint(-hi, hi + 1, (N, dp), device=DEV, generator=g).float()
    if kind == "crowded":                              # the nearest ones all lie in the last columns
        c[max(0, N - 200):] *= 0.0
        c[max(0, N - 200):, 0] = torch.arange(min(N, 200), device=DEV).float().flip(0)
    if kind == "equal":
        c[:] = c[0]
    d = (q.double() ** 2).sum(1)[:, None] + (c.double() ** 2).sum(1) - 2 * (q.double() @ c.double().T)
    order = torch.argsort(d, dim=1, stable=True)
    for k in sorted({1, 2, 16, 64, 84, 127, 128, 129, 300, 1024}):
        if k > N:
            continue
        probes, got = erq.coarse_probe(q, c, k, with_dist=True)
        assert torch.equal(probes.long(), order[:, :k])
        assert torch.equal(got.double(), d.gather(1, order[:, :k]))
