"""What the online trainers allocate, and when: the first call, whatever its size, leaves later ones nothing to
allocate (they can be captured into a graph), and a model whose first call is captured is trained all the same
where that never needed scratch."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
from workloads import make_workload  # noqa: E402

from test_gpu_online_batched import clustered  # noqa: E402
from test_gpu_parity import dev_u32, make_ctx, rel_err  # noqa: E402


def setup(D, C, N, seed=3):
    wl = make_workload(1, D=D, C=C, F=3, L=2)
    hv, y = clustered(np.random.default_rng(seed), N, D, C)
    return make_ctx(wl), hv, y, dev_u32(hv), torch.from_numpy(y).cuda()


def captured_three_times(call, acc):
    """Rows after three replays of the captured call, each from zero, with eager work in between."""
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        acc.zero_()
        call(acc)
    out = []
    for _ in range(3):
        graph.replay()
        out.append(acc.cpu())
        acc.fill_(7.0)
        torch.cuda.synchronize()
    return out


# (samples, batch) of the first call and of the one captured after it; batch 0: hdc_train_online
@pytest.mark.parametrize("first,then", [((2, 0), (300, 0)), ((300, 0), (2, 0)), ((600, 300), (600, 64)), ((100, 64), (600, 64)),
                                        ((600, 64), (100, 64)), ((600, 8), (20, 8)), ((300, 0), (1, 0))])
@pytest.mark.parametrize("D,C", [(1000, 5), (2000, 20), (40000, 2)])
def test_the_first_call_leaves_nothing_to_allocate(D, C, first, then):
    ctx, hv, y, hvd, yd = setup(D, C, 600)
    if D > 32768 and 0 in (first[1], then[1]):     # one sample a batch, of any number
        first, then = (first[0], first[1] or 1), (then[0], then[1] or 1)

    def call(acc, n, batch):
        if batch:
            ctx.hdc_train_online_batched(hvd[:n], yd[:n], acc, batch, epochs=1, lr=1.0)
        else:
            ctx.hdc_train_online(hvd[:n], yd[:n], acc, epochs=1, lr=1.0)

    acc = torch.zeros((C, D), dtype=torch.float32, device="cuda")
    call(acc, *first)
    n, batch = then
    want = (oracle.train_online_batched(hv[:n], y[:n], D, C, batch, epochs=1, lr=1.0) if batch
            else oracle.train_online(hv[:n], y[:n], D, C, epochs=1, lr=1.0))
    for got in captured_three_times(lambda a: call(a, n, batch), acc):
        assert rel_err(got.numpy(), want) < 1e-4
    ctx.close()


# 13 classes and more (in registers up to 32 at D = 1024, 40 at 2048, 20 at 4096), or 7 and more at large D
@pytest.mark.parametrize("D,C", [(1000, 20), (1024, 32), (600, 40), (2048, 40), (4096, 20), (10000, 7), (16384, 2), (2500, 33)])
def test_a_captured_first_call(D, C):
    ctx, hv, y, hvd, yd = setup(D, C, 40)
    acc = torch.zeros((C, D), dtype=torch.float32, device="cuda")
    replays = captured_three_times(lambda a: ctx.hdc_train_online(hvd, yd, a, epochs=2, lr=0.5), acc)
    want = oracle.train_online(hv, y, D, C, epochs=2, lr=0.5)
    for got in replays:
        assert rel_err(got.numpy(), want) < 1e-4
    acc.zero_()
    ctx.hdc_train_online(hvd, yd, acc, epochs=2, lr=0.5)      # and in blocks afterwards
    assert rel_err(acc.cpu().numpy(), want) < 1e-4
    ctx.close()
