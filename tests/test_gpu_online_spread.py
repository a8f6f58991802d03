"""Online training of more than 1024 samples in blocks of up to 2048, each block's chain spread over a workgroup per 16
samples (csrc/online_spread.hip), per sample and in batches, against the CPU oracle: at the edges of workgroups and blocks,
of the class lists, where batches begin inside a workgroup or end with one, and where predictions are mostly wrong, so that
the workgroups finish a block one after another."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
from workloads import make_workload  # noqa: E402

from test_gpu_online_batched import clustered  # noqa: E402
from test_gpu_online_chain import TOL, blocks_of_256, off  # noqa: E402
from test_gpu_online_wide import labels  # noqa: E402
from test_gpu_parity import dev_u32, make_ctx  # noqa: E402


def train(ctx, hvd, yd, acc, batch, epochs, lr=1.0):
    """One call (batch 0: hdc_train_online); says whether it went in blocks of 2048."""
    ctx.hdc_profile_enable(True)
    if batch:
        ctx.hdc_train_online_batched(hvd, yd, acc, batch, epochs=epochs, lr=lr)
    else:
        ctx.hdc_train_online(hvd, yd, acc, epochs=epochs, lr=lr)
    spread = ctx.hdc_profile_read("online_spread")[1]
    assert not (spread and ctx.hdc_profile_read("online_wide")[1])     # (counts calls in blocks of 256)
    return spread


def goes(C, N, batch):
    """In blocks of 2048: per sample, and where there are enough batches for what a block costs."""
    few = C <= 16
    return batch == 0 or (batch <= 256 and N >= max(1280 if few else 1536, (8 + 5 * -(-N // 2048)) * batch) and (few or batch >= 16))


def want(hv, y, D, C, batch, epochs, lr=1.0, acc=None):
    if batch:
        return oracle.train_online_batched(hv, y, D, C, batch, epochs=epochs, lr=lr, acc=acc)
    return oracle.train_online(hv, y, D, C, epochs=epochs, lr=lr, acc=acc)


# one workgroup more than 1024 samples, edges of a workgroup's 16 samples, of a block and the next; classes at one and two a
# wave and the most of them; small, odd and large D
@pytest.mark.parametrize("batch", [0, 1, 7, 16, 17, 64, 85, 160])
@pytest.mark.parametrize("D,C,N", [(64, 1, 1025), (1000, 2, 1296), (1001, 5, 2047), (2049, 16, 2048), (640, 17, 2049), (640, 32, 2200),
                                   (10000, 6, 2600), (333, 9, 4097)])
def test_long_calls_match_the_oracle(D, C, N, batch):
    rng = np.random.default_rng(D + 10 * C + N)
    hv, y = clustered(rng, N, D, C)
    y[N // 2] = C                                  # out of range: skipped
    hv[N - 1], y[N - 1] = hv[0], y[0]              # the same sample twice
    ctx = make_ctx(make_workload(1, D=D, C=C, F=3, L=2))
    hvd, yd = dev_u32(hv), torch.from_numpy(y).cuda()
    acc = torch.zeros((C, D), dtype=torch.float32, device="cuda")
    for calls in (1, 2):                           # the second call goes on from the rows of the first
        assert train(ctx, hvd, yd, acc, batch, 1, 0.5) == goes(C, N, batch)
        assert off(acc, want(hv, y, D, C, batch, calls, 0.5)) < TOL
    ctx.close()


def packed(rng, N, D, C):
    """clustered() for many dimensions: an eighth of the bits differ from the class's"""
    words = lambda n: rng.integers(0, 1 << 32, (n, (D + 31) // 32), dtype=np.uint32)  # noqa: E731
    y = rng.integers(0, C, N).astype(np.int32)
    hv = words(C)[y] ^ (words(N) & words(N) & words(N))
    if D % 32:
        hv[:, -1] &= np.uint32((1 << (D % 32)) - 1)
    return hv, y


# Slices of more than 512 dimensions' worth of partial sums (D > 10240), squared norms of more than 256 groups (16384), per sample up to D = 32768
# and in batches to 65535, where products reach the limits of 16 bits: equal samples and ones that differ in every bit
@pytest.mark.parametrize("batch", [0, 1, 40])
@pytest.mark.parametrize("D,C,N", [(10241, 3, 1300), (20001, 20, 1600), (32767, 2, 1290), (40000, 2, 1281), (65535, 3, 1300)])
def test_long_calls_of_many_dimensions(D, C, N, batch):
    rng = np.random.default_rng(D)
    hv, y = packed(rng, N, D, C)
    hv[700], y[700] = hv[3], y[3]
    hv[1200], y[1200] = ~hv[5], (y[5] + 1) % C
    hv[1201], y[1201] = ~hv[1199], (y[1199] + 1) % C
    if D % 32:
        hv[:, -1] &= np.uint32((1 << (D % 32)) - 1)
    ctx = make_ctx(make_workload(1, D=D, C=C, F=3, L=2))
    acc = torch.zeros((C, D), dtype=torch.float32, device="cuda")
    assert train(ctx, dev_u32(hv), torch.from_numpy(y).cuda(), acc, batch, 2) == goes(C, N, batch)
    assert off(acc, want(hv, y, D, C, batch, 2)) < TOL
    ctx.close()


# 16384 samples are held at a time, 8192 at the largest D: products are made again every epoch
@pytest.mark.parametrize("D,C,N,batch", [(96, 3, 16384 + 300, 0), (96, 3, 16384 + 300, 100), (65535, 2, 8192 + 40, 25)])
def test_long_calls_of_more_samples_than_are_held(D, C, N, batch):
    hv, y = packed(np.random.default_rng(D), N, D, C)
    ctx = make_ctx(make_workload(1, D=D, C=C, F=3, L=2))
    acc = torch.zeros((C, D), dtype=torch.float32, device="cuda")
    assert train(ctx, dev_u32(hv), torch.from_numpy(y).cuda(), acc, batch, 2)
    assert off(acc, want(hv, y, D, C, batch, 2)) < 1e-5   # n <= 11000: sqrt(n) 2^-23
    ctx.close()


# all samples of one class (its list runs through every row of lanes), hardly any valid, classes in runs
@pytest.mark.parametrize("kind", ["one", "most", "few", "blocks"])
@pytest.mark.parametrize("batch", [0, 40])
@pytest.mark.parametrize("D,C,N", [(1000, 4, 2100), (512, 16, 1500), (512, 20, 2500)])
def test_long_calls_of_uneven_classes(D, C, N, batch, kind):
    rng = np.random.default_rng(D + C + N)
    hv, y = clustered(rng, N, D, C)
    y = labels(kind, rng, y, C)
    ctx = make_ctx(make_workload(1, D=D, C=C, F=3, L=2))
    acc = torch.zeros((C, D), dtype=torch.float32, device="cuda")
    assert train(ctx, dev_u32(hv), torch.from_numpy(y).cuda(), acc, batch, 2)
    assert off(acc, want(hv, y, D, C, batch, 2)) < TOL
    ctx.close()


# Wrong predictions: some (listed beside the right ones), and so many that workgroups go on alone; one to eight classes to a
# row of lanes; batches that fill workgroups, cross them, and several to a workgroup
@pytest.mark.parametrize("flip,wrong", [(0.1, 1.0), (0.1, 0.5), (0.1, 0.2), (0.45, 0.0)])
@pytest.mark.parametrize("batch", [0, 10, 16, 64, 100])
@pytest.mark.parametrize("D,C,N", [(1000, 2, 2048), (999, 6, 3000), (640, 12, 2100), (512, 24, 2100)])
def test_long_calls_of_wrong_predictions(D, C, N, batch, flip, wrong):
    rng = np.random.default_rng(D + 10 * C + N)
    hv, y = clustered(rng, N, D, C, flip)
    y = np.where(rng.random(N) < wrong, rng.integers(0, C, N), y).astype(np.int32)
    ctx = make_ctx(make_workload(1, D=D, C=C, F=3, L=2))
    hvd, yd = dev_u32(hv), torch.from_numpy(y).cuda()
    acc = torch.zeros((C, D), dtype=torch.float32, device="cuda")
    train(ctx, hvd, yd, acc, batch, 1)
    assert off(acc, want(hv, y, D, C, batch, 1)) < TOL
    again = torch.zeros_like(acc)                  # the same bits every time
    train(ctx, hvd, yd, again, batch, 1)
    assert torch.equal(acc, again)
    ctx.close()


def starting_rows(kind, rng, hv, y, D, C):
    """zeros; at random; trained on other labels, of all samples or of half of them"""
    if kind == "zero":
        return np.zeros((C, D), dtype=np.float32)
    if kind == "random":
        return rng.normal(size=(C, D)).astype(np.float32)
    named = (y[:200] + 1) % C
    return oracle.train_online(hv[:200], (named if kind == "other" else np.where(rng.random(200) < 0.5, y[:200], named)).astype(np.int32), D, C, epochs=1, lr=1.0)


# Most predictions change at the second pass, because they are right then: the passes go on
@pytest.mark.parametrize("kind", ["random", "other", "half"])
@pytest.mark.parametrize("batch", [0, 32])
@pytest.mark.parametrize("D,C,N", [(1000, 2, 2000), (1000, 6, 2100), (2000, 20, 2048)])
def test_long_calls_from_rows_that_know_other_labels(D, C, N, batch, kind):
    rng = np.random.default_rng(D + C + N)
    hv, y = clustered(rng, N, D, C)
    start = starting_rows(kind, rng, hv, y, D, C)
    ctx = make_ctx(make_workload(1, D=D, C=C, F=3, L=2))
    acc = torch.from_numpy(start.copy()).cuda()
    assert train(ctx, dev_u32(hv), torch.from_numpy(y).cuda(), acc, batch, 1)
    assert off(acc, want(hv, y, D, C, batch, 1, acc=start.copy())) < TOL
    ctx.close()


def test_rows_that_know_other_labels_take_no_longer_than_zeros():
    D, C, N = 1000, 6, 2000                        # 145 us either way; 480 from such rows if workgroups go on alone
    rng = np.random.default_rng(1)
    hv, y = clustered(rng, N, D, C)
    ctx = make_ctx(make_workload(1, D=D, C=C, F=3, L=2))
    hvd, yd, took = dev_u32(hv), torch.from_numpy(y).cuda(), {}
    for kind in ("zero", "other"):
        start = torch.from_numpy(starting_rows(kind, rng, hv, y, D, C)).cuda()
        took[kind] = []
        for _ in range(8):
            acc, first, last = start.clone(), torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            first.record()
            ctx.hdc_train_online(hvd, yd, acc, epochs=1, lr=1.0)
            last.record()
            torch.cuda.synchronize()
            took[kind].append(first.elapsed_time(last))
    ctx.close()
    assert min(took["other"]) < 2 * min(took["zero"]), took


# With more than 16 classes passes go on, 96 of them (24 classes: 70 are enough; 17 of few dimensions: 110 to 150 would be)
@pytest.mark.parametrize("D,C,N", [(512, 24, 2048), (200, 17, 2100), (64, 18, 2048)])
def test_long_calls_of_many_classes_and_random_labels(D, C, N):
    rng = np.random.default_rng(D + C)
    hv, y = clustered(rng, N, D, C)
    y = rng.integers(0, C, N).astype(np.int32)
    ctx = make_ctx(make_workload(1, D=D, C=C, F=3, L=2))
    hvd, yd, rows = dev_u32(hv), torch.from_numpy(y).cuda(), []
    for _ in range(2):                             # the second call finds the words as the first one found them
        rows.append(torch.zeros((C, D), dtype=torch.float32, device="cuda"))
        assert train(ctx, hvd, yd, rows[-1], 0, 1)
    assert torch.equal(rows[0], rows[1]) and off(rows[0], want(hv, y, D, C, 0, 1)) < TOL
    ctx.close()


# (panels of 256 samples, of 240, 195 and 200 in batches; the last block of one panel)
@pytest.mark.parametrize("batch", [0, 20, 65, 100])
@pytest.mark.parametrize("row,value", [(0, float("nan")), (1, float("inf"))])
@pytest.mark.parametrize("C", [3, 20, 32])
def test_long_calls_from_rows_that_are_not_finite(C, row, value, batch):
    D, N = 200, 2100
    hv, y = clustered(np.random.default_rng(C), N, D, C)
    start = np.random.default_rng(6).normal(size=(C, D)).astype(np.float32)
    start[row, 7] = value
    ctx = make_ctx(make_workload(1, D=D, C=C, F=3, L=2))
    hvd, yd, acc = dev_u32(hv), torch.from_numpy(y).cuda(), torch.from_numpy(start.copy()).cuda()
    assert train(ctx, hvd, yd, acc, batch, 1)
    if batch:    # (against calls of one batch each: the oracle takes class 0 here as well)
        single = torch.from_numpy(start.copy()).cuda()
        for n in range(0, N, batch):
            ctx.hdc_train_online_batched(hvd[n:n + batch], yd[n:n + batch], single, batch, epochs=1, lr=1.0)
        expected = single.cpu().numpy()
    else:
        expected = want(hv, y, D, C, 0, 1, acc=start.copy())
    got, ok = acc.cpu().numpy(), np.isfinite(expected)
    assert np.array_equal(np.isnan(got), np.isnan(expected)) and np.array_equal(got[np.isinf(expected)], expected[np.isinf(expected)])
    assert np.max(np.abs(got[ok] - expected[ok]), initial=0.0) <= TOL * max(1.0, float(np.max(np.abs(expected[ok]), initial=0.0)))
    ctx.close()


@pytest.mark.parametrize("batch", [0, 32])
def test_rows_that_are_not_finite_take_no_longer_than_in_blocks_of_256(batch):
    D, C, N = 500, 6, 2048                         # 4 ms either way; 10 where each sample was added to by all before it
    hv, y = clustered(np.random.default_rng(C), N, D, C)
    hvd, yd, took = dev_u32(hv), torch.from_numpy(y).cuda(), []
    start = torch.full((C, D), 1.0, device="cuda")
    start[1, 7] = float("inf")
    for ctx in (blocks_of_256(make_ctx(make_workload(1, D=D, C=C, F=3, L=2))), make_ctx(make_workload(1, D=D, C=C, F=3, L=2))):
        times = []
        for _ in range(4):
            acc, first, last = start.clone(), torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            first.record()
            if batch:
                ctx.hdc_train_online_batched(hvd, yd, acc, batch, epochs=1, lr=1.0)
            else:
                ctx.hdc_train_online(hvd, yd, acc, epochs=1, lr=1.0)
            last.record()
            torch.cuda.synchronize()
            times.append(first.elapsed_time(last))
        took.append(min(times))
        ctx.close()
    assert took[1] < 1.5 * took[0], took


@pytest.mark.parametrize("wrong", [0.0, 1.0])
def test_long_calls_replayed_from_a_graph(wrong):
    D, C, N = 1000, 5, 2500
    rng = np.random.default_rng(2)
    hv, y = clustered(rng, N, D, C, 0.1)
    y = np.where(rng.random(N) < wrong, rng.integers(0, C, N), y).astype(np.int32)
    ctx = make_ctx(make_workload(1, D=D, C=C, F=3, L=2))
    hvd, yd = dev_u32(hv), torch.from_numpy(y).cuda()
    acc = torch.zeros((C, D), dtype=torch.float32, device="cuda")
    eager = torch.zeros_like(acc)
    ctx.hdc_train_online(hvd[:5], yd[:5], eager, epochs=1, lr=1.0)     # scratch is set up here
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        acc.zero_()
        ctx.hdc_train_online(hvd, yd, acc, epochs=2, lr=1.0)
    for k in range(3):
        hvd.copy_(hvd.roll(17, dims=0))
        yd.copy_(yd.roll(17, dims=0))
        graph.replay()
        eager.zero_()
        ctx.hdc_train_online(hvd, yd, eager, epochs=2, lr=1.0)
        torch.cuda.synchronize()
        assert torch.equal(acc, eager), k
    ctx.close()


@pytest.mark.parametrize("C,N,batch,lr,spread", [
    (2, 1024, 0, 1.0, 0), (2, 1025, 0, 1.0, 1), (32, 2000, 0, 1.0, 1), (33, 2000, 0, 1.0, 0), (3, 2000, 153, 1.0, 1), (3, 2000, 154, 1.0, 0), (3, 1279, 2, 1.0, 0),
    (3, 1280, 2, 1.0, 1), (17, 1535, 16, 1.0, 0), (17, 1536, 16, 1.0, 1), (1, 7168, 256, 1.0, 1), (1, 7167, 256, 1.0, 0), (1, 8000, 257, 1.0, 0),
    (17, 2000, 15, 1.0, 0), (17, 2000, 16, 1.0, 1), (3, 2000, 0, 1e30, 0), (3, 2000, 0, float("nan"), 0)])
def test_which_calls_go_in_blocks_of_2048(C, N, batch, lr, spread):
    ctx = make_ctx(make_workload(1, D=64, C=C, F=3, L=2))
    hvd = torch.zeros((N, ctx.W), dtype=torch.int32, device="cuda")
    yd = torch.zeros(N, dtype=torch.int32, device="cuda")
    assert train(ctx, hvd, yd, torch.zeros((C, 64), dtype=torch.float32, device="cuda"), batch, 1, lr) == spread
    ctx.close()
