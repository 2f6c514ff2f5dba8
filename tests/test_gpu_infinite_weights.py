"""An infinite weight in a job whose depth ends inside a k-step: it reaches the outputs that it belongs to, as the infinity that it makes there."""
import numpy as np
import pytest

from oracle import dense, train
from gpu_util import DevicePool, norm_rel_err
from paper_1902_04610_amd import salus, synth
from test_gpu_kernels import NONE, TOL_BF16_TIGHT
from test_gpu_order_of_sums import forward
from test_gpu_train import TOL_GRAD, TrainJob

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shapes", [
    [(129, 448, 264), (140, 392, 264)],          # 32 x 32 register tiles: the second job takes what the first one takes
    [(257, 384, 1032), (129, 424, 1032)],        # 32 x 64
    [(33, 40, 136)], [(48, 72, 520)] * 9,        # both, up to 128 rows
    [(40, 2504, 320)], [(60, 1064, 776)] * 4,    # deep enough for steps in front of the last ones, which drop nothing
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


@pytest.mark.parametrize("dims, M, lr", [((40, 64, 72), 33, 0.5), ((72, 256, 40), 129, 0.25), ((40, 64, 2504), 33, 0.5)])
def test_infinite_weight_of_the_label(dims, M, lr):
    """Input gradients through 32 x 32 register tiles: an infinite loss whose gradient is an infinity and no NaN."""
    rng = np.random.default_rng(M)
    label, unit = 3, 5
    Wm = [(rng.uniform(0.5, 1.0, dims[:2]) / dims[0]).astype(np.float32), (rng.standard_normal(dims[1:]) / np.sqrt(dims[1])).astype(np.float32)]
    Wm[1][unit, label] = -np.inf
    dp = DevicePool(1 << 22, policy=salus.POLICY_PACK)
    job = TrainJob(dp, dims, M, lr, Wm)
    X, labels = synth.f32_to_bf16_bits(rng.uniform(0.5, 1.0, (M, dims[0])).astype(np.float32)), np.full(M, label, np.int32)
    job.put_batch(X, labels)
    descs, keep = salus.Pool.make_train_descs([job.desc()])
    assert dp.pool.grouped_train_step(descs, stream=dp.stream) == salus.OK
    dp.sync()
    (W, _), _, logits, loss = job.gpu_state()
    dp.close()
    _, _, grads = train.train_step(X, labels, job.Wm, job.Wb, job.lr)
    assert np.isneginf(logits[:, label]).all() and loss == np.inf
    assert np.isneginf(W[:, unit]).all() and np.isneginf(job.Wm[0][:, unit]).all(), W[:4, unit]
    rest = np.arange(dims[1]) != unit
    bound = lr * TOL_GRAD * np.abs(grads[0][:, rest]).max() + 2.0 ** -23 * np.abs(W[:, rest]).max()
    assert np.abs(W - job.Wm[0])[:, rest].max() <= bound
