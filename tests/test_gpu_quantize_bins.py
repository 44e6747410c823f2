"""Algorithm 1 by bins and bounds against the oracle's heap enumeration, at the
edges of the kernel's widths (threads and coordinates per vector) and on rows
whose maximum is hard to bound: exact ties, two scales, outliers, few non-zeros.
Codes must be equal; the factors are FP64 results rounded to FP32 from FP64
sums of another order (at most dp 2^-53 relative), so one FP32 rounding each
side: 2^-23 and a margin.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2409_09913_amd import erq, synth

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

DEV = torch.device("cuda:0")


def hard_rows(dp, seed):
    g = np.random.default_rng(seed)
    x = g.standard_normal((8, dp))
    rows = list(synth.edge_rows(dp, seed=seed).astype(np.float64))
    rows += [x[0], g.laplace(size=dp), x[1] * np.exp(2 * g.standard_normal(dp))]
    rows.append(np.where(np.arange(dp) < dp // 2, x[2], 1e-3 * x[2]))              # two scales
    rows.append(np.where(np.arange(dp) < max(1, dp // 50), x[3], 0.02 * x[3]))     # few large, many small
    rows.append(np.where(np.arange(dp) == dp - 1, 1000.0, x[4]))                   # one outlier
    rows.append(np.where(g.random(dp) < 0.1, x[5], 0.0))                           # sparse
    rows.append(np.sign(x[6]) * 1.7)                                               # every critical value tied
    rows.append(np.where(np.arange(dp) % 2, 0.75, 0.0))                            # tied, maximum at the last level
    rows.append(np.round(2 * x[7]) / 2)                                            # many ties
    return np.asarray(rows, np.float32)


@pytest.mark.parametrize("dp,B", [(64, 5), (256, 4), (320, 8), (512, 2), (576, 6), (768, 4), (768, 5), (832, 3),
                                  (1024, 8), (1088, 5), (1536, 7), (1600, 4), (2048, 5), (2112, 2), (3072, 5)])
def test_quantize_widths_and_hard_rows(dp, B):
    print("quantize bins", dp, B, flush=True)
    r = hard_rows(dp, seed=dp + B)
    want, wfa, wfr, wco = oracle.quantize(r.astype(np.float64), B)
    m = r.shape[0]
    for n in (m, 512, 513, 1024, 1025):          # few vectors: four waves each; more: as few as the width needs
        rr = np.ascontiguousarray(np.tile(r, ((n + m - 1) // m, 1))[:n])
        codes, fa, fr, co = [t.cpu().numpy() for t in erq.quantize(torch.from_numpy(rr).to(DEV), B)]
        at = np.arange(n) % m
        bad = np.nonzero((codes != want[at]).any(1))[0]
        assert bad.size == 0, f"dp={dp} B={B} n={n}: rows {sorted(set((bad % m).tolist()))} differ"
        np.testing.assert_allclose(fa, wfa.astype(np.float32)[at], rtol=2.5e-7, atol=0)
        np.testing.assert_allclose(fr, wfr.astype(np.float32)[at], rtol=4e-7, atol=0)
        np.testing.assert_allclose(co, wco.astype(np.float32)[at], rtol=4e-7, atol=0)


def test_quantize_element_aligned_arrays():
    """Rows that start on a 4-byte and codes that start on a 1-byte boundary."""
    dp, n, B = 320, 37, 4
    x = torch.from_numpy(synth.random_rotated(n, dp, seed=9)).to(DEV)
    want = erq.quantize(x, B)
    buf = torch.empty(n * dp + 1, dtype=torch.float32, device=DEV)
    buf[1:] = x.flatten()
    out = torch.zeros(n * dp + 1, dtype=torch.uint8, device=DEV)
    f = [torch.empty(n, dtype=torch.float32, device=DEV) for _ in range(3)]
    rc = erq.load().erq_quantize(buf[1:].data_ptr(), n, dp, B, None, out[1:].data_ptr(), *[t.data_ptr() for t in f],
                                 torch.cuda.current_stream().cuda_stream)
    assert rc == 0
    assert torch.equal(out[1:].view(n, dp), want[0]) and int(out[0]) == 0
    for a, b in zip(f, want[1:]):
        assert torch.equal(a, b)
