"""GPU parity of the weight update around the rows that a tile requests at once and the edges of its blocks, against the oracle."""
import pytest

import test_gpu_train
from test_gpu_once_and_few import FarPool
from test_gpu_train import run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M", [1, 32, 33, 65, 191])
@pytest.mark.parametrize("dims", [(72, 264, 8), (8, 40, 520)])
def test_updates_of_few_blocks(dims, M):
    """Blocks of 64 x 64: widths below a block, that end inside one and of several."""
    run([(dims, M, 0.05)], steps=1, seed=20 + M)


MANY = 12          # jobs of these widths have more blocks of 64 x 64 than are under way at once
DIMS = (520, 1032, 264)


@pytest.mark.parametrize("M", [1, 33, 64, 88, 89])
def test_updates_of_few_rows(M):
    """Blocks of 32 x 64 up to 88 rows, of 64 x 64 beyond."""
    run([(DIMS, M, 0.05)] * MANY, steps=1, seed=40 + M)


@pytest.mark.parametrize("rows", [[97], [128], [129], [100, 150]])
def test_updates_of_few_rows_with_weights_from_further_away(rows, monkeypatch):
    """Up to a mean of 128 rows; jobs with more rows than a tile requests at once."""
    monkeypatch.setattr(test_gpu_train, "DevicePool", FarPool)
    # rows on either side of 128 have two launches of each forward layer
    run([(DIMS, rows[i % len(rows)], 0.05) for i in range(MANY)], steps=1, seed=31, extra_forward_launches=2 if len(rows) > 1 else 0)


@pytest.mark.parametrize("dims, M", [((520, 1800, 776), 33), ((1320, 1288, 392), 80), ((72, 2016, 1024), 64)])
def test_rows_of_blocks_that_end_with_a_partial_one(dims, M):
    """8, 4, 6, 2 blocks of 32 x 64 x 4 side by side, the last one a few columns wide or nearly whole."""
    run([(dims, M, 0.05)] * 4, steps=1, seed=70)
