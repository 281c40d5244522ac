"""Register-staged BF16 / FP8 tiles of 128x128 wave blocks, whose chunks follow the
products where they are 16 or more a lane and stage and go under them where they
are fewer: bit for bit the LDS-DMA pipeline's results, as the narrower tiles."""
import pytest

import test_lp_staged_gpu as staged

pytestmark = pytest.mark.gpu

TILES = {1: [(256, 256, 16, 32), (128, 256, 16, 32), (128, 128, 16, 32), (256, 256, 16, 64), (128, 256, 16, 64),
             (128, 128, 16, 128)],
         2: [(256, 256, 16, 64), (256, 128, 16, 64), (128, 128, 16, 64), (256, 256, 16, 128), (128, 128, 16, 256)]}


@pytest.mark.parametrize("dtype", [1, 2])
@pytest.mark.parametrize("ta,tb", [(0, 0), (0, 1), (1, 0), (1, 1)])
def test_odd_rows_equal_padded_rows(gpu, kt, monkeypatch, dtype, ta, tb):
    monkeypatch.setattr(staged, "TILES", TILES)
    staged.test_odd_rows_equal_padded_rows(gpu, kt, dtype, ta, tb)
