"""Online training in blocks of samples (csrc/online_chain.hip) against the CPU oracle, at the sizes where
the blocks, sub-blocks, classes per wave and dimension groups change."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
from paper_2206_04746_amd import binding  # noqa: E402
from workloads import make_workload  # noqa: E402

from test_gpu_online_batched import clustered  # noqa: E402
from test_gpu_parity import dev_u32, make_ctx  # noqa: E402

# A block's cosines leave out the fp32 rounding of the updates made since it began: u updates that name a row,
# each off by at most 2^-24 of its elements, and the signs of those errors as good as random, so a cosine by about
# sqrt(u) 2^-24 (measured, rows from zero: up to 3e-7 over D = 33 to 4096, 1 to 16 classes, samples 2 to 35 %
# from their prototype; u 2^-24 at the very most).  A weight moves by as much.  An element is a sum of n
# such weights of random sign: sqrt(n) 3e-7, whatever its own size (an element next to zero by as much as a large
# one: hence the bound against the largest), which against rows of size sqrt(n) is 3e-7.  Seven times that.
TOL = 2e-6


def blocks_of_256(ctx):
    """The context as it is where the scratch of longer blocks could not be had."""
    assert getattr(binding.lib, "_ZN3hdc21reserve_online_blocksEPNS_12hdc_ctx_implE")(ctx._h) == 0
    return ctx


def off(acc, want):
    return float(np.max(np.abs(acc.cpu().numpy() - want)) / np.max(np.abs(want)))


# a few samples (fewer than a batch's dozen go sample by sample: test_gpu_online_short.py); one sub-block and its
# edges; one block and its edges; several blocks; classes at one, two and four to a wave; one class; odd D, the
# smallest and largest D
SHAPES = [(1000, 5, 6), (1000, 5, 7), (2049, 3, 63), (2049, 3, 64), (10000, 6, 65), (1000, 2, 255), (1000, 16, 256),
          (1001, 17, 257), (640, 32, 300), (640, 33, 300), (512, 64, 600), (100, 1, 300), (65535, 2, 70), (63, 2, 130)]


@pytest.mark.parametrize("batch", [0, 1, 7, 64, 85])   # 0: hdc_train_online
@pytest.mark.parametrize("D,C,N", SHAPES)
def test_blocks_match_the_oracle(D, C, N, batch):
    rng = np.random.default_rng(D + 100 * C + N)
    wl = make_workload(1, D=D, C=C, F=3, L=2)
    hv, y = clustered(rng, N, D, C)
    y[N // 2] = C                                  # out of range: skipped
    hv[N - 1], y[N - 1] = hv[0], y[0]              # the same sample twice
    ctx = make_ctx(wl)
    hvd, yd = dev_u32(hv), torch.from_numpy(y).cuda()
    acc = torch.zeros((C, D), dtype=torch.float32, device="cuda")
    for calls in (1, 2):                           # the second call goes on from the rows of the first
        if batch:
            ctx.hdc_train_online_batched(hvd, yd, acc, batch, epochs=2, lr=0.5)
            want = oracle.train_online_batched(hv, y, D, C, batch, epochs=2 * calls, lr=0.5)
        else:
            ctx.hdc_train_online(hvd, yd, acc, epochs=2, lr=0.5)
            want = oracle.train_online(hv, y, D, C, epochs=2 * calls, lr=0.5)
        assert off(acc, want) < TOL
    ctx.close()


# Samples close to their prototypes (weights next to zero, and the roundings of a row's updates alike), and rows that
# are large to begin with.  What a cosine leaves out is at most half a unit of every element for each of the u updates of
# the row in the block and the one before, u 2^-24 of the row, and a weight moves by as much; N weights of random sign, and
# an element's own rounding.  (u <= 512, of which the classes share: 256 is asked for.)
@pytest.mark.parametrize("batch", [0, 20])
@pytest.mark.parametrize("size", [0.0, 1.0, 1e3, 1e6])
@pytest.mark.parametrize("D,C,flip", [(64, 1, 0.05), (100, 2, 0.02), (1024, 5, 0.02), (1000, 17, 0.1), (4096, 3, 0.35)])
def test_similar_samples_and_large_rows(D, C, flip, size, batch):
    rng = np.random.default_rng(D + C)
    N = 700
    hv, y = clustered(rng, N, D, C, flip)
    start = (size * rng.normal(size=(C, D))).astype(np.float32)
    ctx = make_ctx(make_workload(1, D=D, C=C, F=3, L=2))
    acc = torch.from_numpy(start.copy()).cuda()
    if batch:
        ctx.hdc_train_online_batched(dev_u32(hv), torch.from_numpy(y).cuda(), acc, batch, epochs=1, lr=1.0)
        want = oracle.train_online_batched(hv, y, D, C, batch, epochs=1, lr=1.0, acc=start)
    else:
        ctx.hdc_train_online(dev_u32(hv), torch.from_numpy(y).cuda(), acc, epochs=1, lr=1.0)
        want = oracle.train_online(hv, y, D, C, epochs=1, lr=1.0, acc=start)
    ctx.close()
    assert np.max(np.abs(acc.cpu().numpy() - want)) <= np.sqrt(N) * 256 * 2.0 ** -24 + 2 * np.spacing(np.abs(want).max())


@pytest.mark.parametrize("batch", [0, 16])
def test_bits_past_the_last_dimension_are_ignored(batch):
    D, C, N = 1001, 4, 300
    hv, y = clustered(np.random.default_rng(4), N, D, C)
    dirty = hv.copy()
    dirty[::3, -1] |= np.uint32(0xffffffff) << np.uint32(D % 32)
    ctx = make_ctx(make_workload(1, D=D, C=C, F=3, L=2))
    yd = torch.from_numpy(y).cuda()
    rows = []
    for h in (hv, dirty):
        acc = torch.zeros((C, D), dtype=torch.float32, device="cuda")
        if batch:
            ctx.hdc_train_online_batched(dev_u32(h), yd, acc, batch, epochs=2, lr=1.0)
        else:
            ctx.hdc_train_online(dev_u32(h), yd, acc, epochs=2, lr=1.0)
        rows.append(acc.cpu())
    assert torch.equal(rows[0], rows[1])
    ctx.close()


NAN, INF = float("nan"), float("inf")


# rows that are no numbers or infinite from the start, and weights that get there in the middle of a block
@pytest.mark.parametrize("batch", [0, 24])
@pytest.mark.parametrize("row,value,lr", [(0, NAN, 1.0), (2, NAN, 1.0), (0, INF, 1.0), (1, -INF, 0.5), (-1, NAN, 1.0), (1, 0.0, INF),
                                          (1, 0.0, NAN), (0, 0.0, -INF)])
@pytest.mark.parametrize("C", [3, 20, 40])
def test_rows_and_weights_that_are_not_finite(C, row, value, lr, batch):
    D, N = 200, 300
    hv, y = clustered(np.random.default_rng(5), N, D, C)
    start = np.random.default_rng(6).normal(size=(C, D)).astype(np.float32)
    if value != 0.0:
        start[row if row >= 0 else slice(None), 7] = value
    ctx = make_ctx(make_workload(1, D=D, C=C, F=3, L=2))
    hvd, yd, acc = dev_u32(hv), torch.from_numpy(y).cuda(), torch.from_numpy(start.copy()).cuda()
    if batch:    # (against calls of one batch each, which do not go in blocks: the oracle takes class 0 here as well)
        ctx.hdc_train_online_batched(hvd, yd, acc, batch, epochs=1, lr=lr)
        single = torch.from_numpy(start.copy()).cuda()
        for n in range(0, N, batch):
            ctx.hdc_train_online_batched(hvd[n:n + batch], yd[n:n + batch], single, batch, epochs=1, lr=lr)
        want = single.cpu().numpy()
    else:
        ctx.hdc_train_online(hvd, yd, acc, epochs=1, lr=lr)
        want = oracle.train_online(hv, y, D, C, epochs=1, lr=lr, acc=start.copy())
    got = acc.cpu().numpy()
    assert np.array_equal(np.isfinite(got), np.isfinite(want)) and np.array_equal(np.isnan(got), np.isnan(want))
    ok = np.isfinite(want)
    assert np.array_equal(got[np.isinf(want)], want[np.isinf(want)])
    assert np.max(np.abs(got[ok] - want[ok]), initial=0.0) <= TOL * max(1.0, float(np.max(np.abs(want[ok]), initial=0.0)))
    ctx.close()


@pytest.mark.parametrize("C,longer", [(3, True), (3, False), (35, True)])
def test_more_samples_than_are_held_at_a_time(C, longer):
    D, N = 96, 16384 + 300                         # the sample products of 16384 rows are held at a time
    rng = np.random.default_rng(1)
    wl = make_workload(1, D=D, C=C, F=3, L=2)
    hv, y = clustered(rng, N, D, C)
    ctx = make_ctx(wl) if longer else blocks_of_256(make_ctx(wl))
    hvd, yd = dev_u32(hv), torch.from_numpy(y).cuda()
    ctx.hdc_profile_enable(True)
    for batch in (8, 60):
        acc = torch.zeros((C, D), dtype=torch.float32, device="cuda")
        ctx.hdc_train_online_batched(hvd, yd, acc, batch, epochs=2, lr=1.0)
        assert ctx.hdc_profile_read("online_spread")[1] == (longer and C <= 32)
        assert off(acc, oracle.train_online_batched(hv, y, D, C, batch, epochs=2, lr=1.0)) < 1e-5   # n <= 11000: sqrt(n) 2^-23
    ctx.close()


def test_blocks_replayed_from_a_graph():
    D, C, N = 10000, 6, 600
    rng = np.random.default_rng(2)
    wl = make_workload(1, D=D, C=C, F=3, L=2)
    hv, y = clustered(rng, N, D, C)
    ctx = make_ctx(wl)
    hvd, yd = dev_u32(hv), torch.from_numpy(y).cuda()
    acc = torch.zeros((C, D), dtype=torch.float32, device="cuda")
    eager = torch.zeros_like(acc)
    ctx.hdc_train_online(hvd, yd, eager, epochs=1, lr=1.0)     # scratch and attributes are set up here
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        acc.zero_()
        ctx.hdc_train_online(hvd, yd, acc, epochs=1, lr=1.0)
    for k in range(3):
        hvd.copy_(hvd.roll(17, dims=0))
        yd.copy_(yd.roll(17, dims=0))
        graph.replay()
        eager.zero_()
        ctx.hdc_train_online(hvd, yd, eager, epochs=1, lr=1.0)
        torch.cuda.synchronize()
        assert torch.equal(acc, eager), k
    ctx.close()


# samples, batch (0: hdc_train_online) -> entries of the counters online, online_fwd, online_bwd; a call in batches
# that goes in blocks has as many of each as it has blocks, one that does not has none of the first
@pytest.mark.parametrize("D,C,N,batch,blocks", [
    (1000, 5, 600, 0, 0), (1000, 5, 600, 8, 3), (1000, 5, 32, 8, 1), (1000, 5, 24, 8, None), (1000, 5, 600, 86, None),
    (1000, 1, 510, 85, None), (1000, 1, 1020, 42, None), (1000, 1, 1024, 32, 4), (20000, 1, 1020, 42, 5), (1000, 17, 510, 85, None),
    (10000, 17, 510, 85, 2), (1000, 8, 510, 85, 2), (4000, 33, 1020, 85, None), (4000, 33, 1024, 64, 4), (1000, 65, 600, 8, None),
    (65535, 3, 1020, 85, 4)])
def test_which_calls_go_in_blocks_and_what_the_counters_say(D, C, N, batch, blocks):
    ctx = make_ctx(make_workload(1, D=D, C=C, F=3, L=2))
    hvd = torch.zeros((N, ctx.W), dtype=torch.int32, device="cuda")
    yd = torch.zeros(N, dtype=torch.int32, device="cuda")
    acc = torch.zeros((C, D), dtype=torch.float32, device="cuda")
    ctx.hdc_profile_enable(True)
    if batch:
        ctx.hdc_train_online_batched(hvd, yd, acc, batch, epochs=1, lr=1.0)
    else:
        ctx.hdc_train_online(hvd, yd, acc, epochs=1, lr=1.0)
    (ms, n), (fwd_ms, fwd), (bwd_ms, bwd) = (ctx.hdc_profile_read(k) for k in ("online", "online_fwd", "online_bwd"))
    if not batch:
        assert (n, fwd, bwd) == (1, 0, 0) and ms > 0
    elif blocks:
        assert (n, fwd, bwd) == (blocks, blocks, blocks) and min(ms, fwd_ms, bwd_ms) > 0
    else:
        batches = -(-N // batch)
        assert n == 0 and fwd == batches and bwd >= batches and min(fwd_ms, bwd_ms) > 0
    ctx.close()
