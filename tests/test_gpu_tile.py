"""The tiled product at the edges of its tiles and of its dispatch: every tile height
(64 to 256 rows in steps of 32), one and two node-row tiles, whole rounds of
256-column tiles followed by narrower ones and narrow tiles alone, ragged rows
and columns, one to three 64-deep steps, and bias groups below, at and above
16 rows.  Past the tiles' 32-bit ranges: the kernels with 64-bit addresses."""
import pytest
import torch

from paper_2608_13524_amd import dartree as D
from tests.gpu_util import device, say
from tests.test_gpu_kernels import check_project_bf16

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows,vocab,hidden,group", [
    # 65 .. 256 rows: one node-row tile of 96, 128, 160, 192, 224, 256 rows;
    # past 65536 columns whole rounds, then the remainder in narrow tiles
    (65, 66000, 64, 7), (96, 65537, 128, 16), (97, 70001, 64, 97), (129, 65601, 192, 25), (161, 83001, 64, 17),
    (193, 65900, 128, 15), (225, 71003, 64, 32), (256, 66049, 64, 64),
    # two node-row tiles, ragged in the second; two bias groups within 16 rows
    (257, 40001, 128, 19), (300, 50257, 64, 25), (511, 34001, 64, 73),
    # 17..64 rows: tiles of 64 rows below 65536 columns, and above with K no multiple of 128 from 33 rows on
    (17, 20001, 128, 4), (32, 8192, 64, 32), (33, 66001, 192, 11), (64, 50257, 128, 16), (50, 70003, 320, 13),
    # <= 16 rows: the pair kernel from 28672 columns, the stream kernel below; one and several pairs of
    # 64 k a wave; 17..64 rows on both sides of rows x columns = 2^18
    (16, 24576, 128, 4), (9, 24575, 128, 3), (16, 30001, 384, 16),
    (4, 28672, 128, 1), (3, 28671, 256, 2), (1, 33000, 4224, 1), (5, 33000, 2176, 2), (20, 13107, 128, 5), (20, 13108, 128, 5),
    # 33..64 rows past the Infinity Cache below 65536 columns: the sweep
    (40, 33000, 4224, 8), (17, 65535, 2176, 8),
    # fewer tiles than compute units: one tile size by cost (96 to 256 rows, 64 to 256 columns)
    (1024, 5121, 1024, 64), (2048, 5120, 256, 512), (1024, 4096, 128, 16), (1000, 16000, 64, 125), (130, 16385, 64, 13),
    (65, 5, 64, 1), (70, 64, 128, 3), (100, 257, 320, 33), (250, 2049, 192, 50), (700, 513, 64, 100),
])
def test_project_tile_edges(rows, vocab, hidden, group):
    check_project_bf16(rows, vocab, hidden, group, pad=1)


@pytest.mark.parametrize("rows,vocab,hidden,group", [
    # outputs on both sides of a tile's 32-bit range: 256 rows at 2^22 columns, fewer rows later
    (256, (1 << 22) - 1, 64, 64), (256, 1 << 22, 64, 64), (257, (1 << 22) + 1, 64, 100), (96, 11184811, 64, 16),
    (40, 26843601, 64, 7),
    # hidden sizes past a tile's operand range
    (65, 130, (1 << 20) + 64, 9), (129, 5, (1 << 20) + 128, 129),
])
def test_project_past_32_bit_ranges(rows, vocab, hidden, group):
    """Small whole numbers: every fp32 sum is exact, so every output is compared for equality."""
    dev = device()
    g = torch.Generator(device=dev).manual_seed(rows)
    whole = lambda shape: torch.randint(-2, 3, shape, generator=g, device=dev, dtype=torch.int8)
    x, U = whole((rows, hidden)).to(torch.bfloat16), whole((vocab, hidden)).to(torch.bfloat16)
    bias = whole(((rows + group - 1) // group, vocab)).float()
    z = torch.full((rows, vocab), 0.5, dtype=torch.float32, device=dev)
    nws = D.project_workspace_size(D.BF16, rows, vocab, hidden)
    ws = torch.empty(nws, dtype=torch.uint8, device=dev) if nws else None
    say(f"project bf16 rows={rows} vocab={vocab} hidden={hidden} (range)")
    D.project(D.BF16, x, U, bias, vocab, z, group, ws)
    row_group = torch.arange(rows, device=dev) // group
    step = 1 << 19
    for n in range(0, vocab, step):
        want = x.float() @ U[n:n + step].float().t() + bias[row_group, n:n + step]
        assert torch.equal(z[:, n:n + step], want), n
    del x, U, bias, z
    torch.cuda.empty_cache()


@pytest.mark.parametrize("vocab,hidden", [(28671, 2560), (28672, 2560), (50257, 4096), (70000, 1280), (5000, 640)])
def test_project_up_to_16_rows_keep_their_bits(vocab, hidden):
    """A row's outputs are the same bits whatever number of rows (up to 16) it comes with."""
    dev = device()
    g = torch.Generator(device=dev).manual_seed(vocab)
    x = torch.tanh(torch.randn(16, hidden, generator=g, device=dev) * 1.4).to(torch.bfloat16)
    U = (torch.randn(vocab, hidden, generator=g, device=dev) * 0.02).to(torch.bfloat16)
    bias = torch.randn(1, vocab, generator=g, device=dev)
    whole = torch.empty(16, vocab, device=dev)
    say(f"project bf16 1 to 16 rows, vocab={vocab} hidden={hidden} (bits)")
    D.project(D.BF16, x, U, bias, 0, whole, 16)
    for rows in (1, 4, 5, 8, 15):
        z = torch.empty(rows, vocab, device=dev)
        D.project(D.BF16, x[:rows].contiguous(), U, bias, 0, z, rows)
        assert torch.equal(z, whole[:rows]), rows


@pytest.mark.parametrize("rows,vocab,hidden,pieces", [
    (20, 16000, 4096, 16), (64, 16000, 4096, 16), (40, 50257, 2560, 16), (64, 5000, 2560, 16), (20, 60001, 4096, 16),
    (64, 60001, 4096, 16), (8, 50257, 2560, 8), (40, 70003, 2624, 16),
])
def test_project_partial_sums(rows, vocab, hidden, pieces):
    """Up to 64 rows against middle-length matrices add K up in partial sums.
    A chain of n additions of terms of one size rounds partial sums whose mean square is half the final one's:
    a variance of u^2 / 3 each (u = 2^-24) makes n u^2 / 6 of the result's square, twice that for the products of
    32 terms that MFMA rounds inside too.  p chains of n / p and the p additions of their sums: (2 n / p + p) u^2 / 6.
    (One chain of 128 products is 2.8 times above this bound at 16 pieces, 4 chains 1.03 times at 8.)"""
    dev = device()
    g = torch.Generator(device=dev).manual_seed(vocab)
    x = torch.tanh(torch.randn(rows, hidden, generator=g, device=dev) * 1.4).to(torch.bfloat16)
    U = (torch.randn(vocab, hidden, generator=g, device=dev) * 0.02).to(torch.bfloat16)
    bias = torch.zeros(1, vocab, device=dev)
    z = torch.empty(rows, vocab, device=dev)
    say(f"project bf16 rows={rows} vocab={vocab} hidden={hidden} (partial sums)")
    D.project(D.BF16, x, U, bias, 0, z, rows)
    want = x.double() @ U[:4096].double().t()
    err = ((z[:, :4096].double() - want).norm() / want.norm()).item()
    assert err < 2.0 ** -24 * ((2 * hidden / 32 / pieces + pieces) / 6) ** 0.5, err
