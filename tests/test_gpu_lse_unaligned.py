"""log-softmax and top-k of rows that start at any multiple of 4 bytes: odd
vocabularies and a z off the 16-byte grid, in every regime of rows (streamed
segments, segments held in registers, whole rows) and at every remainder."""
import numpy as np
import pytest
import torch

import oracle.dartree_ref as R
from paper_2608_13524_amd import dartree as D
from tests.gpu_util import device, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows,vocab,k,T,offset", [
    (1, 1, 1, 0.0, 3), (3, 5, 5, 1.0, 1), (2, 4097, 8, 0.7, 0), (16, 50257, 16, 1.0, 2),
    (17, 8193, 8, 1.0, 0), (40, 20003, 32, 0.0, 1), (100, 8191, 4, 0.7, 3), (20, 600001, 8, 1.0, 0),
    (512, 4099, 8, 1.0, 0), (513, 16386, 16, 0.0, 1), (600, 8192, 8, 1.0, 2),
])
def test_lse_topk_unaligned(rows, vocab, k, T, offset):
    rng = np.random.default_rng(rows + vocab + offset)
    z = rng.normal(0, 2, size=(rows, vocab)).astype(np.float32)
    z[0, -1] = z[0].max() + 1   # the best of a row in its ragged end
    dev = device()
    buf = torch.full((rows * vocab + 8,), 1e30, device=dev)   # neighbours that would win any comparison
    zd = buf[offset:offset + rows * vocab].view(rows, vocab)
    zd.copy_(torch.from_numpy(z))
    lse = torch.empty(rows, device=dev)
    lp = torch.empty(rows, k, device=dev)
    ids = torch.empty(rows, k, dtype=torch.int32, device=dev)
    ws = torch.empty(max(D.lse_topk_workspace_size(rows, vocab, k), 1), dtype=torch.uint8, device=dev)
    say(f"lse_topk unaligned rows={rows} vocab={vocab} k={k} offset={offset}")
    D.lse_topk(zd, k, T, lse, lp, ids, ws)
    torch.cuda.synchronize()
    tau = T if T > 0 else 1.0
    z64 = z.astype(np.float64)
    m = z64.max(axis=1)
    want_lse = m / tau + np.log(np.exp((z64 - m[:, None]) / tau).sum(axis=1))
    want_ids = np.stack([R.topk_ids(z64[r], k) for r in range(rows)])
    assert np.array_equal(ids.cpu().numpy(), want_ids)
    # fp32 sums of at most 600001 terms in partial sums of a few hundred: below 2e-6 relative, as the aligned test
    assert np.allclose(lse.cpu().numpy(), want_lse, rtol=2e-6, atol=2e-5)
    want_lp = np.take_along_axis(R.log_softmax(z64, tau), want_ids.astype(np.int64), axis=1)
    assert np.abs(lp.cpu().numpy() - want_lp).max() < 2e-5


@pytest.mark.parametrize("rows,vocab,finite,offset", [
    # whole rows: threads whose first 32 values are all masked
    (600, 9001, 600, 0), (512, 9000, 300, 0), (520, 20003, 8, 1),
    # streamed segments of few rows: masked threads and wholly masked segments
    (2, 600001, 300, 0), (16, 300000, 5000, 0),
    # segments held in registers
    (20, 8001, 40, 0), (40, 20003, 8, 2),
])
def test_lse_topk_masked(rows, vocab, finite, offset):
    """Rows whose values past the first `finite` are -inf: the normaliser and the best of what is left."""
    k = 8
    rng = np.random.default_rng(rows + vocab)
    z = np.full((rows, vocab), -np.inf, dtype=np.float32)
    z[:, :finite] = rng.normal(0, 2, size=(rows, finite))
    dev = device()
    buf = torch.full((rows * vocab + 8,), 1e30, device=dev)
    zd = buf[offset:offset + rows * vocab].view(rows, vocab)
    zd.copy_(torch.from_numpy(z))
    lse = torch.empty(rows, device=dev)
    lp = torch.empty(rows, k, device=dev)
    ids = torch.empty(rows, k, dtype=torch.int32, device=dev)
    ws = torch.empty(max(D.lse_topk_workspace_size(rows, vocab, k), 1), dtype=torch.uint8, device=dev)
    say(f"lse_topk masked rows={rows} vocab={vocab} finite={finite}")
    D.lse_topk(zd, k, 1.0, lse, lp, ids, ws)
    torch.cuda.synchronize()
    z64 = z[:, :finite].astype(np.float64)
    m = z64.max(axis=1)
    want_lse = m + np.log(np.exp(z64 - m[:, None]).sum(axis=1))
    want_ids = np.argsort(-z64, axis=1, kind="stable")[:, :k]
    assert np.array_equal(ids.cpu().numpy(), want_ids)
    assert np.allclose(lse.cpu().numpy(), want_lse, rtol=2e-6, atol=2e-5)
    want_lp = np.take_along_axis(z64, want_ids, axis=1) - want_lse[:, None]
    assert np.abs(lp.cpu().numpy() - want_lp).max() < 2e-5
