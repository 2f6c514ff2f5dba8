"""An infinite weight in a job whose depth ends inside a k-step: it reaches the outputs that it belongs to, as the infinity that it makes there."""
import numpy as np
import pytest

from oracle import dense
from gpu_util import norm_rel_err
from paper_1902_04610_amd import synth
from test_gpu_kernels import NONE, TOL_BF16_TIGHT
from test_gpu_order_of_sums import forward

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shapes", [
    [(129, 448, 264), (140, 392, 264)],          # 32 x 32 register tiles: the second job takes what the first one takes
    [(257, 384, 1032), (129, 424, 1032)],        # 32 x 64
    [(33, 40, 136)], [(48, 72, 520)] * 9,        # both, up to 128 rows
])
def test_infinite_weight(shapes):
    """Lanes past the last k-row read the first ones again, times zero."""
    rng = np.random.default_rng(7)
    jobs = []
    for M, K, N in shapes:
        W = synth.f32_to_bf16_bits((rng.standard_normal((K, N)) / np.sqrt(K)).astype(np.float32))
        W[3, 5] = 0x7f80                         # +inf in a k-row and a column of the first ones
        jobs.append((synth.f32_to_bf16_bits(rng.uniform(0.5, 1.0, (M, K)).astype(np.float32)), W))
    for (X, W), Y in zip(jobs, forward(jobs)):
        assert np.isposinf(Y[:, 5]).all(), Y[:4, 5]
        W = W.copy()
        W[3, 5] = 0
        rest = np.arange(W.shape[1]) != 5
        assert norm_rel_err(Y[:, rest], dense.dense_bf16(X, W, NONE)[:, rest]) < TOL_BF16_TIGHT
