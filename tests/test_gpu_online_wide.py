"""Per-sample online training with the blocks walked as a whole and a block's row updates beside the next block's
chain (csrc/online_chain.hip, up to 16 classes and D = 32767, from 129 samples on, 128 (C - 2) + 1 in all epochs, two thirds of a block from 5 classes on, of all blocks from 9 on) against
the CPU oracle: where the order of the products changes, at the edges of sub-blocks and blocks, and where calls leave it.  The
contexts have no scratch for longer blocks, in which calls of more than 1024 samples go otherwise (test_gpu_online_spread.py)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
from workloads import make_workload  # noqa: E402

from test_gpu_online_batched import clustered  # noqa: E402
from test_gpu_online_chain import TOL, blocks_of_256, off  # noqa: E402
from test_gpu_parity import dev_u32, make_ctx  # noqa: E402


def labels(kind, rng, y, C):
    """as drawn; of one class throughout (its list goes through five waves); one class in ten samples out of eleven;
    almost none valid; one class a sub-block; at random (predictions mostly wrong)"""
    n = np.arange(len(y))
    return {"drawn": y, "one": np.full_like(y, C - 1), "most": np.where(n % 11, 0, y), "few": np.where(n % 29, -1, y),
            "blocks": (n // 64 % C).astype(np.int32), "random": rng.integers(0, C, len(y)).astype(np.int32)}[kind]


def train(ctx, hv, y, acc, epochs, lr):
    """One call; says whether it went in blocks that are walked as a whole."""
    ctx.hdc_profile_enable(True)
    ctx.hdc_train_online(dev_u32(hv), torch.from_numpy(y).cuda(), acc, epochs=epochs, lr=lr)
    assert ctx.hdc_profile_read("online")[1] == 1
    return ctx.hdc_profile_read("online_wide")[1]


@pytest.mark.parametrize("C,D,N,epochs,lr,wide", [
    (2, 64, 128, 9, 1.0, 0), (2, 64, 129, 1, 1.0, 1), (1, 64, 129, 1, 1.0, 1), (16, 64, 896, 2, 1.0, 0), (16, 64, 1793, 1, 1.0, 1),
    (8, 64, 256, 3, 1.0, 0), (8, 64, 256, 4, 1.0, 1), (4, 64, 257, 1, 1.0, 1), (5, 64, 170, 9, 1.0, 0), (5, 64, 171, 9, 1.0, 1), (8, 64, 257, 3, 1.0, 1),
    (9, 64, 341, 9, 1.0, 0), (9, 64, 342, 9, 1.0, 1), (9, 64, 513, 9, 1.0, 1), (17, 64, 4000, 1, 1.0, 0), (3, 32767, 129, 1, 1.0, 1), (3, 32768, 129, 1, 1.0, 0),
    (3, 64, 300, 1, 0.9e30, 1), (3, 64, 300, 1, 1e30, 0), (3, 64, 300, 1, float("nan"), 0)])
def test_which_calls_go_in_blocks_walked_as_a_whole(C, D, N, epochs, lr, wide):
    ctx = blocks_of_256(make_ctx(make_workload(1, D=D, C=C, F=3, L=2)))
    hv, y = np.zeros((N, ctx.W), np.uint32), np.zeros(N, np.int32)
    assert train(ctx, hv, y, torch.zeros((C, D), dtype=torch.float32, device="cuda"), epochs, lr) == wide
    ctx.close()


# one more than two sub-blocks, edges of three and four, of a block and the next; classes at one and two a wave (four
# and two rows a group) and past them; smallest D, odd D, the largest and one more
@pytest.mark.parametrize("kind", ["drawn", "one", "most", "few", "blocks", "random"])
@pytest.mark.parametrize("D,C,N", [(1000, 4, 129), (1000, 8, 171), (1001, 9, 192), (1000, 1, 193), (2049, 3, 257), (640, 16, 513), (640, 16, 342), (10000, 6, 600),
                                   (512, 17, 300), (32, 2, 300), (32767, 2, 300), (32768, 2, 300)])
def test_blocks_as_a_whole_match_the_oracle(D, C, N, kind):
    rng = np.random.default_rng(D + 10 * C + N)
    hv, y = clustered(rng, N, D, C)
    y = labels(kind, rng, y, C)
    ctx = blocks_of_256(make_ctx(make_workload(1, D=D, C=C, F=3, L=2)))
    acc = torch.zeros((C, D), dtype=torch.float32, device="cuda")
    epochs = max(2, 128 * (C - 2) // N + 1)        # with fewer samples in all they go by sub-blocks
    for calls in (1, 2):                           # the second call goes on from the rows of the first
        assert train(ctx, hv, y, acc, epochs, 0.5) == (C <= 16 and D <= 32767)
        assert off(acc, oracle.train_online(hv, y, D, C, epochs=epochs * calls, lr=0.5)) < TOL
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
    ctx = blocks_of_256(make_ctx(make_workload(1, D=D, C=C, F=3, L=2)))
    acc = torch.zeros((C, D), dtype=torch.float32, device="cuda")
    assert train(ctx, hv, y, acc, 2, 1.0)
    assert off(acc, oracle.train_online(hv, y, D, C, epochs=2, lr=1.0)) < TOL
    ctx.close()


# Rows that are no numbers or infinite from the start, at one and two classes a wave: every block of these is walked
# sample by sample, the later ones beside the row updates of the block before
@pytest.mark.parametrize("row,value", [(0, float("nan")), (-1, float("nan")), (0, float("inf")), (1, float("-inf")), (slice(None), float("nan"))])
@pytest.mark.parametrize("C,N", [(2, 700), (8, 800), (9, 1100), (16, 1900)])
def test_rows_that_are_not_finite(C, N, row, value):
    D = 200
    hv, y = clustered(np.random.default_rng(C), N, D, C)
    start = np.random.default_rng(6).normal(size=(C, D)).astype(np.float32)
    start[row, 7] = value
    ctx = blocks_of_256(make_ctx(make_workload(1, D=D, C=C, F=3, L=2)))
    acc = torch.from_numpy(start.copy()).cuda()
    assert train(ctx, hv, y, acc, 1, 1.0)
    got, want = acc.cpu().numpy(), oracle.train_online(hv, y, D, C, epochs=1, lr=1.0, acc=start.copy())
    assert np.array_equal(np.isnan(got), np.isnan(want)) and np.array_equal(got[np.isinf(want)], want[np.isinf(want)])
    ok = np.isfinite(want)
    assert np.array_equal(np.isfinite(got), ok)
    assert np.max(np.abs(got[ok] - want[ok]), initial=0.0) <= TOL * max(1.0, float(np.max(np.abs(want[ok]), initial=0.0)))
    ctx.close()


def test_more_samples_than_are_held_at_a_time():
    D, C, N = 96, 3, 16384 + 300                   # 64 blocks are held at a time
    hv, y = clustered(np.random.default_rng(1), N, D, C)
    ctx = blocks_of_256(make_ctx(make_workload(1, D=D, C=C, F=3, L=2)))
    acc = torch.zeros((C, D), dtype=torch.float32, device="cuda")
    assert train(ctx, hv, y, acc, 2, 1.0)
    assert off(acc, oracle.train_online(hv, y, D, C, epochs=2, lr=1.0)) < 1e-5   # n <= 6000: sqrt(n) 2^-23
    ctx.close()
