"""The tiled product at the edges of its tiles and of its dispatch: every tile height
(64 to 256 rows in steps of 32), one and two node-row tiles, whole rounds of
256-column tiles followed by narrower ones and narrow tiles alone, ragged rows
and columns, one to three 64-deep steps, and bias groups below, at and above
16 rows."""
import pytest

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
    # <= 16 rows: the pair kernel from 24576 columns, the stream kernel below; 17..64 rows on both
    # sides of rows x columns = 2^18
    (16, 24576, 128, 4), (9, 24575, 128, 3), (16, 30001, 384, 16), (20, 13107, 128, 5), (20, 13108, 128, 5),
    # 33..64 rows past the Infinity Cache below 65536 columns: the sweep
    (40, 33000, 4224, 8),
    # fewer tiles than compute units: narrow tiles alone
    (65, 5, 64, 1), (70, 64, 128, 3), (100, 257, 320, 33), (250, 2049, 192, 50), (700, 513, 64, 100),
])
def test_project_tile_edges(rows, vocab, hidden, group):
    check_project_bf16(rows, vocab, hidden, group, pad=1)
