"""Cosine inference, whose dot products of sample bits with real class rows go by digits of 8 bits from a size on (csrc/row_dots.hip),
against numpy in extended precision.  Below that size: few samples, classes and dimensions of every kind.  By digits: class counts on
both sides of 4, 8 and 16 to a tile of columns and of a chunk, dimensions at the edges of a slice and of more slices than partial sums,
samples at the edges of a wave's and a block's; rows whose elements differ by many orders of magnitude, which digits do not hold,
subnormal ones, rows of zeros, and rows that are not finite; dot products that are equal."""
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


def by_digits(D, C, N):
    """Whether a call of up to 8192 queries takes its dot products by digits."""
    return N <= 8192 and N * C * D >= (12e6 if C <= 8 else 60e6)


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


@pytest.mark.parametrize("kind", ["normal", "orders", "spikes", "subnormal"])
@pytest.mark.parametrize("D,C,N", [(512, 3, 7900), (513, 4, 6001), (1023, 5, 2400), (1025, 8, 1537), (1024, 9, 6600), (2049, 16, 1900), (2049, 17, 1801),
                                   (5121, 33, 400), (11265, 3, 360), (20481, 2, 300), (40000, 2, 151), (300001, 2, 21)])
def test_cosines_by_digits_are_rounded_once(D, C, N, kind):
    assert by_digits(D, C, N)
    rng = np.random.default_rng(D + C + N)
    acc = rng.normal(size=(C, D))
    if kind == "orders":
        acc[1:] *= np.exp(8 * rng.normal(size=(C - 1, D)))      # beside a row that digits hold
    if kind == "spikes":
        acc[:, 700::1500] *= 1e9                                # in some slices
    if kind == "subnormal":
        acc *= 1e-40
    got, pred, want = cosines(D, C, N, acc.astype(np.float32), rng)
    assert np.all(np.abs(got - want) <= 2.0 ** -24 * np.abs(want) * (1 + 1e-6) + 1e-14)
    assert np.all(np.take_along_axis(want, pred[:, None].astype(np.int64), 1)[:, 0] >= want.max(1) - 1e-13)


@pytest.mark.parametrize("C,N", [(3, 70), (7, 70), (18, 70), (3, 1601), (7, 701), (18, 1400)])
def test_rows_of_zeros_and_rows_that_are_not_finite(C, N):
    D = 2500
    rng = np.random.default_rng(1)
    assert by_digits(D, C, N) == (N > 70)
    acc = rng.normal(size=(C, D)).astype(np.float32)
    acc[0] = 0.0
    acc[1, 1030] = np.inf
    acc[2, 3] = np.nan
    got, _, want = cosines(D, C, N, acc, rng)
    rest = [0] + list(range(3, C))
    assert np.all(np.abs(got[:, rest] - want[:, rest]) <= 2.0 ** -24 * np.abs(want[:, rest]) * (1 + 1e-6) + 1e-14)
    assert np.all(np.isnan(got[:, 1])) and np.all(np.isnan(got[:, 2]))      # infinite dot products over infinite norms


# w's last bits 2 and 6 of 8: halfway between two multiples of the upper digits' unit.  +w and -w have digits that are not the
# negatives of one another; a dot product is w times a whole number all the same, and equal ones go to the lowest class.
@pytest.mark.parametrize("last", [2, 6, 4, 7])
@pytest.mark.parametrize("C", [2, 7, 18])
def test_equal_dot_products_go_to_the_lowest_class(C, last):
    D, N = 1000, 8000 if C < 9 else 4000
    rng = np.random.default_rng(10 * C + last)
    w = np.float32((0xD2D680 + last) * 2.0 ** -24)
    signs = rng.integers(0, 2, (C, D)).astype(np.int32) * 2 - 1
    signs[:, 0] = signs[:, 1:].prod(axis=1)                 # (rows that differ in an odd number of places never tie)
    hv = rng.integers(0, 1 << 32, (N, (D + 31) // 32), dtype=np.uint32)
    hv[:, -1] &= np.uint32((1 << (D % 32)) - 1)
    queries = 2 * np.unpackbits(hv.view(np.uint8), axis=1, bitorder="little")[:, :D].astype(np.int32) - 1
    dots = (queries.astype(np.float64) @ signs.T.astype(np.float64)).astype(np.int32)
    assert by_digits(D, C, N)
    assert (np.sort(dots, axis=1)[:, -1] == np.sort(dots, axis=1)[:, -2]).sum() > 100
    ctx = make_ctx(make_workload(1, D=D, C=C, F=3, L=2))
    pred = torch.empty(N, dtype=torch.int32, device="cuda")
    cos = torch.empty((N, C), dtype=torch.float32, device="cuda")
    ctx.hdc_search_cosine(dev_u32(hv), torch.from_numpy(w * signs.astype(np.float32)).cuda(), pred, cos)
    torch.cuda.synchronize()
    ctx.close()
    assert np.array_equal(pred.cpu().numpy(), dots.argmax(1))


# The odd classes' rows are the even ones' with neighbours exchanged and negated, the queries differ in every pair of neighbours:
# such dot products and squared norms are equal in pairs, whatever the order they are summed in, as long as the sums are exact: elements of
# 24 bits in one binade and in eight
@pytest.mark.parametrize("binades", [1, 8])
@pytest.mark.parametrize("C", [2, 6, 18])
def test_mirrored_rows_have_equal_dot_products(C, binades):
    D, N = 1024 + 64, 8000 if C < 9 else 4000
    rng = np.random.default_rng(C + binades)
    rows = np.empty((C, D), dtype=np.float32)
    rows[::2] = np.ldexp(rng.integers(1 << 23, 1 << 24, (C // 2, D)) * rng.choice([-1.0, 1.0], (C // 2, D)),
                         rng.integers(-binades, 0, (C // 2, D))).astype(np.float32)
    rows[1::2] = -rows[::2].reshape(C // 2, D // 2, 2)[:, :, ::-1].reshape(C // 2, D)
    assert by_digits(D, C, N)
    first = rng.integers(0, 2, (N, D // 2), dtype=np.uint8)
    hv = np.packbits(np.stack([first, 1 - first], axis=2).reshape(N, D), axis=1, bitorder="little").view(np.uint32)
    ctx = make_ctx(make_workload(1, D=D, C=C, F=3, L=2))
    pred = torch.empty(N, dtype=torch.int32, device="cuda")
    cos = torch.empty((N, C), dtype=torch.float32, device="cuda")
    ctx.hdc_search_cosine(dev_u32(hv), torch.from_numpy(rows).cuda(), pred, cos)
    torch.cuda.synchronize()
    ctx.close()
    got = cos.cpu().numpy()
    assert np.array_equal(got[:, ::2].view(np.int32), got[:, 1::2].view(np.int32))
    assert np.all(pred.cpu().numpy() % 2 == 0)
