"""Shared candidate sets where their threshold can go wrong: as many groups as
candidates and four times as many, groups of one value and ragged ones, values
that share their 16 leading bits, infinite and zero values of both signs, the
best values all in one group, finite values in fewer groups than candidates
(a masked vocabulary: more and fewer finite values than candidates), and ties
below and above the cap of the radix fallback.  Bit for bit against a full
sort."""
import numpy as np
import pytest
import torch

from paper_2608_13524_amd import dartree as D
from tests.gpu_util import device, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows,vocab,K,kind", [
    (1, 1, 1, "normal"), (3, 256, 256, "normal"), (2, 300, 256, "normal"), (2, 1027, 256, "ties"),
    (5, 50257, 64, "normal"), (2, 151937, 200, "close"), (3, 16385, 5, "close"), (2, 70001, 64, "one group"),
    (2, 20011, 33, "infinite"), (2, 40000, 64, "zeros"), (2, 9000, 100, "constant"), (1, 1 << 20, 256, "normal"),
    (2, 5000, 64, "constant"), (65, 4099, 16, "normal"),
    # long groups (few candidates), read by a block; every group flagged
    (2, 151937, 1, "normal"), (2, 50257, 3, "normal"), (1, 1 << 20, 1, "ties"), (3, 16389, 1, "normal"),
    (2, 30011, 1, "zeros"), (2, 1030, 257 - 1, "normal"), (3, 5, 5, "normal"), (2, 16386, 1, "one group"),
    (2, 151936, 64, 32000), (2, 151937, 64, 100), (3, 50257, 64, 64), (2, 50257, 100, 63), (2, 3000, 64, 200),
    (2, 3000, 64, 10), (1, 20000, 256, 0), (2, 4096, 1, 1),
])
def test_candidate_sets_threshold(rows, vocab, K, kind):
    g = np.random.default_rng(vocab + K)
    x = g.standard_normal((rows, vocab)).astype(np.float32) * 2
    if kind == "ties":
        x = np.round(x)
    elif kind == "close":   # one bf16 step apart at most: every group has the same code or its neighbour
        x = (1.0 + g.random((rows, vocab)) * 2.0 ** -8).astype(np.float32)
    elif kind == "one group":
        at = vocab // 3
        x[:, at:at + 2 * K] += 50
    elif kind == "infinite":
        x[:, ::7] = -np.inf
        x[0, 11] = x[1, vocab - 1] = np.inf
    elif kind == "zeros":
        x = np.where(g.random((rows, vocab)) < 0.5, np.float32(0.0), np.float32(-0.0))
        x[:, ::3] = -1
    elif kind == "constant":
        x[:] = -3.5
    elif isinstance(kind, int):   # only `kind` values in a row are finite, in one range of ids
        at = (vocab - kind) // 3
        x[:, :at] = x[:, at + kind:] = -np.inf
    dev = device()
    xd = torch.from_numpy(np.ascontiguousarray(x)).to(dev)
    ids = torch.full((rows, K), -7, dtype=torch.int32, device=dev)
    ws = torch.full((max(D.candidate_sets_workspace_size(rows, vocab, K), 16),), 0x7F, dtype=torch.uint8, device=dev)
    say(f"candidate sets rows={rows} V={vocab} K={K} {kind}")
    D.candidate_sets(xd, K, ids, ws)
    torch.cuda.synchronize()
    got = ids.cpu().numpy()
    for r in range(rows):
        want = np.lexsort((np.arange(vocab), -x[r].astype(np.float64)))[:K]
        assert np.array_equal(got[r], want), (r, got[r][:10], want[:10])
