"""Row passes at the edges of the rule for their chunks: series of up to 64 rows
and of more, short rows and long, one chunk that fills less and more than four
fifths of the device; against numpy as in test_gpu_row_chunks.
"""

import pytest

import test_gpu_row_chunks as chunks

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("series,K,N", [(600, 40, 2060), (818, 13, 2052), (820, 13, 1100), (700, 64, 16), (700, 65, 16),
                                        (1500, 40, 16), (1300, 40, 256), (1300, 40, 257), (1100, 16, 1500), (17, 64, 255),
                                        (60, 100, 3)])
def test_rows_of_every_chunk(dev, series, K, N):
    chunks.test_every_row_of_every_chunk(dev, series, K, N)
