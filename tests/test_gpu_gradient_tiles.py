"""GPU parity of input gradients on either side of the line between 32 x 32 register tiles and the ring, against the oracle."""
import pytest

from test_gpu_train import run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims, M", [
    ((40, 8, 24), 33), ((136, 520, 2056, 72), 64), ((72, 1000, 264, 40), 129), ((72, 264, 2120), 300),      # one of 32 x 32 per compute unit at most
    ((72, 2056, 264), 127), ((72, 2056, 264), 129),                                                         # 260 and 325 of them
])
def test_input_gradients_of_few_tiles(dims, M):
    run([(dims, M, 0.05)], steps=1, seed=60)
