"""The vector encoders for calls beyond a few samples (csrc/encode.hip, csrc/encode_sparse.hip) against the CPU oracle: the
waves of a block sharing a sample and a sample to a wave, one, two and four samples at a time, all plane counts, full
and compact tables, no varying dimension at all, ragged D and F.  The level vectors are unrelated to one another, so
the contraction does not take these models, and the counters tell that the one-launch kernel for a few samples did
not either."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
from workloads import make_workload, pack_bits_lsb  # noqa: E402

from test_gpu_parity import make_ctx  # noqa: E402


def model(D, F, L, N, vary, u8):
    """A workload whose level vectors are random in the first `vary` of a random order of the dimensions (0: equal)."""
    rng = np.random.default_rng([D, F, L, vary])
    wl = make_workload(3 if u8 else 2, seed=D + F, D=D, F=F, L=L, n_train=N)
    lv = np.repeat(rng.integers(0, 2, size=(1, D), dtype=np.uint8), L, axis=0)
    cols = rng.permutation(D)[:vary]
    if cols.size:
        lv[:, cols] = rng.integers(0, 2, size=(L, cols.size), dtype=np.uint8)
        lv[1, cols] = lv[0, cols] ^ 1
    wl.level = pack_bits_lsb(lv)
    x = rng.integers(0, 256, size=(N, F), dtype=np.uint8) if u8 else rng.uniform(-1.1, 1.1, size=(N, F)).astype(np.float32)
    x[rng.random(x.shape) < 0.6] = 0 if u8 else -1.0          # most features in bin 0
    if not u8:
        x[0, 0], x[-1, -1] = np.nan, 1.0
    return wl, x


# D, F, L, N, dimensions that vary, bytes
CASES = [
    # a sample shared by sixteen waves (up to 256 sample-slices): 8 (compact), 10, 12 and 16 planes
    (20000, 196, 16, 101, 1000, True), (2048, 1000, 16, 256, 2048, False), (2048, 3000, 9, 91, 2048, False), (2049, 5000, 7, 5, 2049, False),
    # by eight waves (up to 2048): the same, and level slices of more than 128 rows
    (10000, 196, 16, 400, 10000, True), (4097, 1001, 200, 300, 4097, False), (2048, 3001, 9, 300, 2048, False), (1000, 5000, 2, 300, 1000, False),
    (33, 31, 16, 1024, 33, False), (1, 1, 2, 2000, 1, False), (31, 2, 2, 1025, 31, False),
    # a sample to a wave, one, two and four at a time
    (2049, 16, 16, 1100, 2049, True), (2048, 17, 256, 2500, 2048, False), (1000, 100, 100, 5121, 1000, True), (320, 15, 50, 12289, 320, False),
    (64, 1, 2, 13000, 64, False), (96, 625, 200, 5200, 96, True), (64, 2500, 5, 2300, 64, False), (40, 4225, 64, 2100, 40, True),
    # compact tables: a few words vary, one does, none does
    (10000, 33, 16, 2000, 3000, False), (4097, 64, 256, 3000, 40, True), (1000, 3, 7, 2048, 1, False), (777, 36, 5, 1500, 0, True),
    (500, 24, 8, 70000, 0, False),
]


@pytest.mark.parametrize("D,F,L,N,vary,u8", CASES)
def test_vector_encoders_bit_exact(D, F, L, N, vary, u8):
    wl, x = model(D, F, L, N, vary, u8)
    ctx = make_ctx(wl)
    compact = 4 * vary <= 3 * D
    assert ctx.hdc_encoded_words() == ((vary + 31) // 32 if compact else ctx.W)
    xd = torch.from_numpy(x).cuda()
    want = oracle.encode(x, wl.D, wl.L, wl.item, wl.level, wl.tie, wl.lo, wl.scale)
    for sparse in (False, True):
        hv = torch.full((N, ctx.W), -1, dtype=torch.int32, device="cuda")
        ctx.hdc_profile_enable(True)
        (ctx.hdc_encode_sparse if sparse else ctx.hdc_encode)(xd, hv)
        launches = {k: ctx.hdc_profile_read(k)[1] for k in ("encode", "quantize", "encode_contract", "encode_wide")}
        ctx.hdc_profile_enable(False)
        chunks = -(-N // 65536)
        assert launches == dict(encode=chunks if vary else 0, quantize=chunks, encode_contract=0, encode_wide=0), sparse
        assert np.array_equal(hv.cpu().numpy().view(np.uint32), want), sparse
    ctx.close()
