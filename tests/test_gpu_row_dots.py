"""Dot products of sample bits with real class rows by digits of 8 bits (csrc/row_dots.hip), through cosine inference, against
numpy in extended precision: class counts on both sides of 4, 8 and 16 to a tile of columns and of a chunk, dimensions at the
edges of a slice and of more slices than ten, samples at the edges of a wave's and a block's; rows whose elements differ by many
orders of magnitude, subnormal ones, rows of zeros, and rows that are not finite."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from workloads import make_workload  # noqa: E402

from test_gpu_parity import dev_u32, make_ctx  # noqa: E402


def cosines(D, C, N, acc, rng):
    W = (D + 31) // 32
    hv = rng.integers(0, 1 << 32, (N, W), dtype=np.uint32)
    if D % 32:
        hv[:, -1] &= np.uint32((1 << (D % 32)) - 1)
    ctx = make_ctx(make_workload(1, D=D, C=C, F=3, L=2))
    pred = torch.empty(N, dtype=torch.int32, device="cuda")
    cos = torch.empty((N, C), dtype=torch.float32, device="cuda")
    ctx.hdc_search_cosine(dev_u32(hv), torch.from_numpy(acc).cuda(), pred, cos)
    torch.cuda.synchronize()
    ctx.close()
    signs = 2 * np.unpackbits(hv.view(np.uint8), axis=1, bitorder="little")[:, :D].astype(np.longdouble) - 1
    rows = acc.astype(np.longdouble)
    with np.errstate(all="ignore"):
        norm = np.sqrt((rows * rows).sum(1)) * np.sqrt(np.longdouble(D))
        want = np.where(norm > 0, (signs @ rows.T) / norm, 0)
    return cos.cpu().numpy(), pred.cpu().numpy(), want


# The fp64 norm's sum of D squares is off by sqrt(D) 2^-53 as a rule, the dot product by less, and the result is rounded to fp32 once.
@pytest.mark.parametrize("kind", ["normal", "orders", "spikes", "subnormal"])
@pytest.mark.parametrize("D,C,N", [(1, 1, 1), (31, 2, 15), (1023, 4, 16), (1024, 5, 17), (1025, 8, 127), (512, 9, 128), (513, 16, 129),
                                   (2049, 17, 300), (10000, 6, 2947), (11265, 3, 40), (5121, 33, 70), (40000, 2, 33), (1000, 6, 20000)])
def test_cosines_are_rounded_once(D, C, N, kind):
    rng = np.random.default_rng(D + C + N)
    acc = rng.normal(size=(C, D))
    if kind == "orders":
        acc *= np.exp(8 * rng.normal(size=(C, D)))
    if kind == "spikes":
        acc[:, ::97] *= 1e9
    if kind == "subnormal":
        acc *= 1e-40
    got, pred, want = cosines(D, C, min(N, 3000 if D > 2000 else N), acc.astype(np.float32), rng)
    assert np.all(np.abs(got - want) <= 2.0 ** -24 * np.abs(want) * (1 + 1e-6) + 1e-14)
    assert np.all(np.take_along_axis(want, pred[:, None].astype(np.int64), 1)[:, 0] >= want.max(1) - 1e-13)


def test_rows_of_zeros_and_rows_that_are_not_finite():
    D, N = 2500, 70
    rng = np.random.default_rng(1)
    for C in (3, 7, 18):
        acc = rng.normal(size=(C, D)).astype(np.float32)
        acc[0] = 0.0
        acc[1, 1030] = np.inf
        acc[2, 3] = np.nan
        got, _, want = cosines(D, C, N, acc, rng)
        rest = [0] + list(range(3, C))
        assert np.all(np.abs(got[:, rest] - want[:, rest]) <= 2.0 ** -24 * np.abs(want[:, rest]) * (1 + 1e-6) + 1e-14)
        assert np.all(np.isnan(got[:, 1])) and np.all(np.isnan(got[:, 2]))      # infinite dot products over infinite norms
