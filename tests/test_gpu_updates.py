"""GPU parity of the weight update around the rows that a tile requests at once and the edges of its blocks, against the oracle."""
import pytest

import test_gpu_train
from test_gpu_once_and_few import FarPool
from test_gpu_train import run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M", [1, 32, 33, 64, 65, 96, 97, 128, 129, 191])
@pytest.mark.parametrize("dims", [(72, 264, 8), (8, 40, 520)])
def test_updates_of_up_to_191_rows(dims, M):
    """Widths below a block, that end inside one and of several; blocks of 32 x 64 up to 64 rows, of 64 x 64 beyond."""
    run([(dims, M, 0.05)], steps=1, seed=20 + M)


@pytest.mark.parametrize("rows", [[65], [128], [97, 40, 33], [20, 17, 300]])
def test_updates_with_weights_from_further_away(rows, monkeypatch):
    """Blocks of 32 x 64 up to a mean of 128 rows, one job with more than are requested at once."""
    monkeypatch.setattr(test_gpu_train, "DevicePool", FarPool)
    dims = (136, 264, 72)
    # 17 - 32, 33 - 128 and more rows take different launches of the forward layers and the input gradient
    extra = {1: 0, 3: 0}[len(rows)] if 300 not in rows else 3
    run([(dims, m, 0.05) for m in rows], steps=1, seed=31, extra_forward_launches=extra)
