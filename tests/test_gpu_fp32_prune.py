"""The fp32 product at the edges of its blocks, and the prune where its
selection can go wrong: ties at the threshold (all, some or none of the tied
nodes kept), more nodes than the registers hold, one-node levels, scores of
both signs and zeros of both signs."""
import numpy as np
import pytest
import torch

import oracle.dartree_ref as R
from paper_2608_13524_amd import dartree as D
from paper_2608_13524_amd import workloads as W
from tests.gpu_util import device, say, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows,vocab,hidden,group", [
    (1, 1, 1, 1), (1, 17, 64, 1), (2, 33, 63, 2), (4, 16, 65, 1), (5, 47, 130, 2), (8, 1000, 192, 8), (9, 15, 7, 4),
    (17, 257, 100, 5),
])
def test_project_fp32_edges(rows, vocab, hidden, group):
    rng = np.random.default_rng(rows * 100 + hidden)
    x = rng.normal(0, 1, size=(rows, hidden)).astype(np.float32)
    U = rng.normal(0, 0.05, size=(vocab, hidden)).astype(np.float32)
    bias = rng.normal(0, 3, size=((rows + group - 1) // group, vocab)).astype(np.float32)
    z = torch.empty(rows, vocab, dtype=torch.float32, device=device())
    say(f"project fp32 rows={rows} vocab={vocab} hidden={hidden}")
    D.project(D.FP32, to_dev(x), to_dev(U), to_dev(bias), vocab, z, group)
    torch.cuda.synchronize()
    x64, U64 = x.astype(np.float64), U.astype(np.float64)
    ref = bias[np.arange(rows) // group].astype(np.float64) + x64 @ U64.T
    # fp32 accumulation of `hidden` products (one rounding each in the fused chain) and the bias add
    bound = 1.01 * (hidden + 4) * 2.0 ** -24 * (np.abs(x64) @ np.abs(U64).T) + 2.0 ** -23 * np.abs(ref) + 1e-12
    assert (np.abs(z.cpu().numpy() - ref) <= bound).all()


@pytest.mark.parametrize("rows,vocab,hidden,group", [
    (65537, 32769, 1, 4096),      # 2^31 outputs and more: two launches, a block row cut between them
    (1, (1 << 28) + 37, 1, 1),    # the same by the columns of one row
])
def test_project_fp32_past_one_launch(rows, vocab, hidden, group):
    """Small whole numbers: every sum is exact."""
    dev = device()
    g = torch.Generator(device=dev).manual_seed(rows)
    whole = lambda shape: torch.randint(-9, 10, shape, generator=g, device=dev, dtype=torch.int8).float()
    x, U, bias = whole((rows, hidden)), whole((vocab, hidden)), whole(((rows + group - 1) // group, vocab))
    z = torch.full((rows, vocab), 0.5, dtype=torch.float32, device=dev)
    say(f"project fp32 rows={rows} vocab={vocab} hidden={hidden} (launches)")
    D.project(D.FP32, x, U, bias, vocab, z, group)
    for m in range(0, rows, group):
        want = x[m:m + group] * U[:, 0] + bias[m // group]
        assert torch.equal(z[m:m + group], want), m
    del x, U, bias, z, want
    torch.cuda.empty_cache()


@pytest.mark.parametrize("batch,L,Wd,k,B,grid", [
    (2, 5, 16, 4, 20, 1.0),      # one score everywhere: the order is depth, slot
    (3, 8, 32, 8, 100, 0.5),     # a few distinct scores: part of a tied group
    (2, 16, 64, 8, 512, 2.0),
    (1, 11, 1500, 2, 1400, 0.25),  # levels above 1024 nodes, more than the registers hold
    (2, 20, 200, 6, 3000, 0.0),  # no ties
    (4, 64, 1, 1, 40, 0.0),      # a chain
    (2, 3, 8, 2, 14, 0.0),       # the whole supertree
])
def test_prune_threshold(batch, L, Wd, k, B, grid):
    rng = np.random.default_rng(L * 1000 + Wd)
    sizes, n = [], 1
    for _ in range(L):
        n = min(Wd, n * k)
        sizes.append(n)
    tok = np.zeros((L, batch, Wd), np.int32)
    par = np.zeros((L, batch, Wd), np.int32)
    sco = np.zeros((L, batch, Wd), np.float32)
    levels = []
    for q in range(batch):
        lv, prev = [], np.full(1, 6.0, np.float32)   # scores fall through zero
        for d, nd in enumerate(sizes):
            pp = rng.integers(0, len(prev), size=nd)
            tt = rng.choice(50000, size=nd, replace=False)
            drop = rng.exponential(1.0, nd)
            drop = np.floor(drop / grid) * grid if grid else drop
            s = (prev[pp] - drop).astype(np.float32)
            if grid and d == 0:
                s[:] = prev[0]
            s[(s == 0) & (rng.random(nd) < 0.5)] = np.float32(-0.0)
            tok[d, q, :nd], par[d, q, :nd], sco[d, q, :nd] = tt, pp, s
            lv.append(R.Level(token=tt.astype(np.int64), parent=pp.astype(np.int64), score=s.astype(np.float64)))
            prev = s
        levels.append(lv)
    cfg = W.Config("prune", batch=batch, vocab=50000, hidden=64, depth=L, width=Wd, branch=k, budget=B,
                   temperature=0.0, precision=W.FP32, seed=0)
    out = D.DeviceTree.alloc(batch, B, device())
    say(f"prune_levels batch={batch} L={L} W={Wd} B={B} grid={grid}")
    D.prune_levels(D.Params.of(cfg), to_dev(tok), to_dev(par), to_dev(sco), out)
    torch.cuda.synchronize()
    got = out.host()
    for q in range(batch):
        t, pa, de, s, m, n = R.emit_tree(levels[q], R.prune(levels[q], B), B)
        assert got["num_nodes"][q] == n
        assert np.array_equal(got["tokens"][q], t) and np.array_equal(got["parents"][q], pa)
        assert np.array_equal(got["depths"][q], de) and np.array_equal(got["mask"][q], m)
        assert np.array_equal(got["scores"][q].astype(np.float64), s)
