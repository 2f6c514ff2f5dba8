"""GPU parity of the weight update around the rows that it requests at once and the edges of its blocks, against the oracle."""
import pytest

from test_gpu_train import run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M", [1, 32, 33, 65, 96, 97, 128, 129, 191])
@pytest.mark.parametrize("dims", [(72, 264, 8), (8, 40, 520)])
def test_updates_of_up_to_191_rows(dims, M):
    """Widths below a block, that end inside one and of several."""
    run([(dims, M, 0.05)], steps=1, seed=20 + M)
