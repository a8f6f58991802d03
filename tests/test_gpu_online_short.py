"""Calls of a few samples of hdc_train_online (csrc/online.hip, sample by sample) and of a few more (blocks)
against the CPU oracle: every kernel variant at its largest class count and dimension, on both sides of the number
of steps up to which it is taken, from zero rows and from trained ones, with wrong predictions."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
from workloads import make_workload  # noqa: E402

from test_gpu_online_batched import clustered  # noqa: E402
from test_gpu_online_chain import TOL, off  # noqa: E402
from test_gpu_parity import dev_u32, make_ctx  # noqa: E402

# classes, dimensions, most steps the walk by samples takes there
LDS = [(1, 1024, 14), (3, 33, 12), (8, 2048, 8), (4, 4096, 11), (2, 3000, 13), (6, 4096, 6), (12, 4096, 6), (9, 1000, 6),
       (1, 10240, 14), (2, 9000, 12), (3, 10240, 6), (6, 10240, 4)]
ONE_LAUNCH = [(2, 16384, 6), (1, 12000, 6), (1, 32768, 2), (20, 4096, 1), (13, 100, 1), (32, 1024, 1), (16, 4000, 2)]
ALWAYS = [(65, 1024, 5), (80, 700, 5), (66, 1025, 3), (100, 512, 3)]     # more than 64 classes, in registers and in memory


@pytest.mark.parametrize("C,D,most", LDS + ONE_LAUNCH + ALWAYS)
def test_a_few_samples(C, D, most):
    rng = np.random.default_rng(C * D)
    hv, y = clustered(rng, most + 1, D, C, flip=0.45)      # (far from their prototypes: mostly wrong predictions)
    ctx = make_ctx(make_workload(1, D=D, C=C, F=3, L=2))
    hvd, yd = dev_u32(hv), torch.from_numpy(y).cuda()
    trained = rng.normal(size=(C, D)).astype(np.float32)
    for n, epochs in {(n, 1) for n in (1, 2, most, most + 1)} | {(1, most), (max(1, most // 2), 2)}:
        for start in (np.zeros_like(trained), trained):
            acc = torch.from_numpy(start.copy()).cuda()
            ctx.hdc_train_online(hvd[:n], yd[:n], acc, epochs=epochs, lr=0.5)
            want, pred, margin = oracle.train_online(hv[:n], y[:n], D, C, epochs=epochs, lr=0.5, acc=start, log=True)
            assert off(acc, want) < TOL, (n, epochs)
            if n > 2 and C > 2 and start.any():
                assert np.any(pred != np.tile(y[:n], epochs))
    ctx.close()


@pytest.mark.parametrize("C,D", [(1, 1000), (4, 3000), (12, 4000), (2, 10000), (6, 10000), (2, 16000), (20, 4000)])
def test_labels_out_of_range_and_calls_in_a_row(C, D):
    rng = np.random.default_rng(D)
    N = 12
    hv, y = clustered(rng, N, D, C)
    y[[1, 5]] = [-1, C]
    ctx = make_ctx(make_workload(1, D=D, C=C, F=3, L=2))
    hvd, yd = dev_u32(hv), torch.from_numpy(y).cuda()
    acc = torch.zeros((C, D), dtype=torch.float32, device="cuda")
    n = 0
    for take in (1, 2, 3, 1, 5):                            # one chain in five calls
        ctx.hdc_train_online(hvd[n:n + take], yd[n:n + take], acc, epochs=1, lr=1.0)
        n += take
    assert n == N and off(acc, oracle.train_online(hv, y, D, C, epochs=1, lr=1.0)) < TOL
    ctx.close()
