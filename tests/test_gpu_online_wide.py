"""Per-sample online training with the blocks walked as a whole and a block's row updates beside the next block's
chain (csrc/online_chain.hip, up to 16 classes and D = 32767, from 129 samples on) against the CPU oracle: where the
order of the products changes, at the edges of sub-blocks and blocks, and where calls leave it."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
from workloads import make_workload  # noqa: E402

from test_gpu_online_batched import clustered  # noqa: E402
from test_gpu_online_chain import TOL, off  # noqa: E402
from test_gpu_parity import dev_u32, make_ctx  # noqa: E402


def labels(kind, rng, y, C):
    """as drawn; of one class throughout (its list goes through five waves); one class in ten samples out of eleven;
    almost none valid; one class a sub-block; at random (predictions mostly wrong)"""
    n = np.arange(len(y))
    return {"drawn": y, "one": np.full_like(y, C - 1), "most": np.where(n % 11, 0, y), "few": np.where(n % 29, -1, y),
            "blocks": (n // 64 % C).astype(np.int32), "random": rng.integers(0, C, len(y)).astype(np.int32)}[kind]


# one more than two sub-blocks, edges of three and four, of a block and the next; classes at one and two a wave (four
# and two rows a group) and past them; smallest D, odd D, the largest and one more
@pytest.mark.parametrize("kind", ["drawn", "one", "most", "few", "blocks", "random"])
@pytest.mark.parametrize("D,C,N", [(1000, 8, 129), (1001, 9, 192), (1000, 1, 193), (2049, 3, 257), (640, 16, 513), (10000, 6, 600),
                                   (512, 17, 300), (32, 2, 300), (32767, 2, 300), (32768, 2, 300)])
def test_blocks_as_a_whole_match_the_oracle(D, C, N, kind):
    rng = np.random.default_rng(D + 10 * C + N)
    hv, y = clustered(rng, N, D, C)
    y = labels(kind, rng, y, C)
    ctx = make_ctx(make_workload(1, D=D, C=C, F=3, L=2))
    hvd, yd = dev_u32(hv), torch.from_numpy(y).cuda()
    acc = torch.zeros((C, D), dtype=torch.float32, device="cuda")
    for calls in (1, 2):                           # the second call goes on from the rows of the first
        ctx.hdc_train_online(hvd, yd, acc, epochs=2, lr=0.5)
        assert off(acc, oracle.train_online(hv, y, D, C, epochs=2 * calls, lr=0.5)) < TOL
    ctx.close()


# Most predictions wrong, or most of them for long: blocks are finished sub-block after sub-block, and the next block begins
# from the squared norms that leaves.  One and two classes a wave, some waves without one, a last block of one to four
# sub-blocks
@pytest.mark.parametrize("flip,wrong", [(0.1, 1.0), (0.1, 0.7), (0.45, 0.0)])
@pytest.mark.parametrize("D,C,N", [(1000, 2, 1025), (1001, 3, 600), (999, 8, 700), (2049, 9, 1100), (640, 12, 1500), (3000, 16, 2000)])
def test_blocks_of_wrong_predictions_match_the_oracle(D, C, N, flip, wrong):
    rng = np.random.default_rng(D + 10 * C + N)
    hv, y = clustered(rng, N, D, C, flip)
    y = np.where(rng.random(N) < wrong, rng.integers(0, C, N), y).astype(np.int32)
    ctx = make_ctx(make_workload(1, D=D, C=C, F=3, L=2))
    acc = torch.zeros((C, D), dtype=torch.float32, device="cuda")
    ctx.hdc_train_online(dev_u32(hv), torch.from_numpy(y).cuda(), acc, epochs=2, lr=1.0)
    assert off(acc, oracle.train_online(hv, y, D, C, epochs=2, lr=1.0)) < TOL
    ctx.close()


def test_more_samples_than_are_held_at_a_time():
    D, C, N = 96, 3, 16384 + 300                   # 64 blocks are held at a time
    hv, y = clustered(np.random.default_rng(1), N, D, C)
    ctx = make_ctx(make_workload(1, D=D, C=C, F=3, L=2))
    acc = torch.zeros((C, D), dtype=torch.float32, device="cuda")
    ctx.hdc_train_online(dev_u32(hv), torch.from_numpy(y).cuda(), acc, epochs=2, lr=1.0)
    assert off(acc, oracle.train_online(hv, y, D, C, epochs=2, lr=1.0)) < 1e-5   # n <= 6000: sqrt(n) 2^-23
    ctx.close()
