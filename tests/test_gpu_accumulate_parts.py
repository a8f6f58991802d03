"""hdc_train_classical of up to 8192 rows (csrc/classical.hip, accumulate_small_kernel): a class's rows split among several
blocks, against sums in numpy: at the edges of the parts and of a wave's rows, of classes that hold all rows, one or none, odd D
and an accumulator that 8-byte stores do not fit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from workloads import make_workload  # noqa: E402

from test_gpu_parity import dev_u32, make_ctx  # noqa: E402


@pytest.mark.parametrize("kind", ["even", "one", "runs"])
@pytest.mark.parametrize("N,C,D", [(1, 1, 64), (256, 1, 65), (257, 1, 2049), (2048, 1, 1000), (8192, 1, 4100), (8191, 2, 1001), (2000, 5, 1024),
                                   (7352, 6, 2100), (513, 2, 31), (3000, 40, 300), (8192, 3, 30000)])
def test_accumulate_in_parts(N, C, D, kind):
    rng = np.random.default_rng(N + C + D)
    W = (D + 31) // 32
    bits = rng.integers(0, 2, (N, D), dtype=np.uint8)
    padded = np.zeros((N, W * 32), dtype=np.uint8)
    padded[:, :D] = bits
    hv = np.packbits(padded, axis=1, bitorder="little").view(np.uint32)
    y = {"even": rng.integers(-1, C + 1, N), "one": np.full(N, C - 1), "runs": np.arange(N) * C // N}[kind].astype(np.int32)
    ctx = make_ctx(make_workload(1, D=D, C=C, F=3, L=2))
    start = rng.integers(-1000, 1000, (C, D), dtype=np.int32)
    store = torch.zeros(C * D + 1, dtype=torch.int32, device="cuda")
    for shift in (0, 1):
        acc = store[shift:shift + C * D].view(C, D)
        acc.copy_(torch.from_numpy(start))
        cn = torch.full((C,), 7, dtype=torch.int64, device="cuda")
        ctx.hdc_train_classical(dev_u32(hv), torch.from_numpy(y).cuda(), acc, cn)
        got, n = acc.cpu().numpy(), cn.cpu().numpy()
        for c in range(C):
            assert np.array_equal(got[c], start[c] + bits[y == c].sum(axis=0, dtype=np.int64)), (c, shift)
            assert n[c] == 7 + int((y == c).sum())
    ctx.close()
