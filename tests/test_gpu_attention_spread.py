"""Tree attention of few rows, whose keys are spread over the waves of a block
and over blocks: one and several shares, one and several steps per wave,
requests that leave shares and waves empty, tree steps that come after context
steps of the same wave, row tiles with remainders, and steps whose last rows
are past the keys.

Tolerance: the weights are rounded to bf16 (relative error <= 2^-9) and their
sum is not, so every element is within 2^-8 max|v| of the exact result, plus
1e-5 for the fp32 sums."""
import numpy as np
import pytest
import torch

from paper_2608_13524_amd import workloads as W
from tests.gpu_util import say
from tests.test_gpu_verify import run_attention

pytestmark = pytest.mark.gpu
SCALE = 1.0 / np.sqrt(128)


def masks_for(b, B, seed):
    """Ancestor-or-self rows of random trees (parents before children); the
    last tenth of the rows are pads that see nothing."""
    g = np.random.default_rng(seed)
    see = np.zeros((b, B, B), bool)
    for q in range(b):
        for i in range(B - B // 10):
            p = g.integers(-1, i)
            if p >= 0:
                see[q, i] = see[q, p]
            see[q, i, i] = True
    bits = np.zeros((b, B, (B + 63) // 64 * 64), np.uint8)
    bits[:, :, :B] = see
    return see, np.packbits(bits, axis=2, bitorder="little").view(np.uint64)


def exact(ai, see, lens, Hq, Hkv):
    f = lambda x: torch.from_numpy(W.bf16_bits_to_fp32(x)).double()
    q, kc, vc, kt, vt = map(f, (ai.q, ai.k_ctx, ai.v_ctx, ai.k_tree, ai.v_tree))
    out = torch.zeros_like(q)
    grp = Hq // Hkv
    for r in range(q.shape[0]):
        n = lens[r]
        k, v = torch.cat([kc[r, :n], kt[r]]), torch.cat([vc[r, :n], vt[r]])
        ok = torch.cat([torch.ones(q.shape[1], n, dtype=torch.bool), torch.from_numpy(see[r])], 1)
        for h in range(Hq):
            s = (q[r, :, h] @ k[:, h // grp].T * SCALE).masked_fill(~ok, -float("inf"))
            out[r, :, h] = torch.nan_to_num(torch.softmax(s, 1)) @ v[:, h // grp]
    return out.numpy()


@pytest.mark.parametrize("b,B,ctx,lens,Hq,Hkv", [
    (4, 64, 2048, [2048, 0, 77, 1999], 32, 8),          # 2 shares, up to 5 steps per wave
    (8, 65, 300, [300, 0, 1, 63, 64, 65, 255, 256], 16, 16),   # 1 share, context and tree steps per wave
    (1, 1500, 0, [0], 1, 1),                            # 24 tree steps in one share
    (2, 600, 400, [400, 130], 2, 1),                    # late mask words
    (1, 8, 20000, [19999], 1, 1),                       # as many shares as steps
    (2, 16, 5000, [5000, 3], 4, 2),                     # a request that leaves most shares empty
    (1, 1, 1, [1], 1, 1),
    (33, 4, 600, list(range(0, 594, 18)), 8, 8),        # 264 blocks of few rows: one block per 256 positions
    (11, 12, 700, list(range(0, 704, 64)), 16, 8),      # 88 blocks of 24 rows: the same
    (11, 25, 300, list(range(0, 308, 28)), 8, 8),       # 25 rows: the spread again
    (10, 24, 300, list(range(0, 310, 31)), 8, 8),       # 80 blocks
    (6, 3, 4100, [4100, 0, 1, 4000, 256, 257], 16, 16),  # 96 blocks, longer contexts
    (33, 12, 0, [0] * 33, 8, 8),                        # the same with the tree's segment alone
    (5, 120, 300, [300, 0, 299, 64, 1], 32, 8),         # 320 blocks of 64 rows: the sweep
])
def test_spread_matches_exact(b, B, ctx, lens, Hq, Hkv):
    say(f"attention spread {b} x {B}, context {ctx}, heads {Hq}/{Hkv}")
    ai = W.make_attention_inputs(b, B, ctx, Hq, Hkv, seed=B + ctx, ctx_len=lens)
    see, mask = masks_for(b, B, seed=B)
    got = run_attention(ai, mask, B, Hq, Hkv, SCALE)
    want = exact(ai, see, lens, Hq, Hkv)
    vmax = max(np.abs(W.bf16_bits_to_fp32(x)).max() for x in (ai.v_ctx, ai.v_tree) if x.size)
    assert np.abs(got - want).max() <= 2.0 ** -8 * vmax + 1e-5


def test_spread_special_values():
    """An infinite value of the last visible position reaches the output as it
    is (rows past it are zeros, not copies of it), and what an earlier call
    left behind does not reach the next."""
    b, B, ctx, Hq, Hkv = 32, 16, 600, 8, 8
    ai = W.make_attention_inputs(b, B, ctx, Hq, Hkv, seed=5, ctx_len=[570] * b)
    see, mask = masks_for(b, B, seed=6)
    say("attention spread, non-finite values")
    full = np.full_like(ai.v_ctx, 0x7FC0)
    keep = ai.v_ctx.copy()
    ai.v_ctx[:] = full
    assert np.isnan(run_attention(ai, mask, B, Hq, Hkv, SCALE)).any()
    ai.v_ctx[:] = keep
    assert np.isfinite(run_attention(ai, mask, B, Hq, Hkv, SCALE)).all()
    ai.v_ctx[:, 569, :, 3] = 0x7F80
    ai.v_ctx[:, 570:] = 0x7FC0   # never read
    got = run_attention(ai, mask, B, Hq, Hkv, SCALE)
    rest = np.delete(got, 3, axis=-1)
    assert np.isfinite(rest).all() and (got[..., 3] == np.inf).all()
