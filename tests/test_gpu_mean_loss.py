"""GPU parity of the mean loss wherever it is taken: in the loss launch, in each kind of update launch, in a launch of its own."""
import pytest

from test_gpu_train import run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("configs", [
    [((40, 64, 64), 64, 0.05)], [((40, 64), 65, 0.05)],          # layers of one width, buffers with too little padding: a launch of its own
    [((40, 72), 17, 0.05)], [((72, 72, 72), 17, 0.05)],          # one width, behind whose gradients there is padding
    [((40, 64, 72), 64, 0.05), ((72, 40), 16, 0.1), ((40, 8), 17, 0.1)], [((40, 64, 64), 64, 0.05), ((40, 64, 72), 40, 0.1)],
    [((72, 40, 264), 600, 0.02), ((72, 264, 40), 513, 0.02)],    # LDS tiles, more rows than are loaded at a time
    [((520, 1032, 264), 40, 0.05)] * 12, [((40, 72, 48, 16), 17 + k % 9, 0.03) for k in range(24)],      # more updates than one launch holds
])
def test_mean_loss(configs):
    rows = [m for _, m, _ in configs]
    run(configs, steps=2, seed=50, extra_forward_launches=int(min(rows) <= 32 < max(rows)),      # one for each side in the first layer
        update_launches=2 if len(configs) * (len(configs[0][0]) - 1) > 64 else 1)
