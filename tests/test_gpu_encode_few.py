"""Encoding of a few samples (csrc/encode_few.hip) against the CPU oracle: last stretch of words partly
filled, one feature, odd and even feature counts around the shares of a block, fp32 and bytes, both block sizes."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
from workloads import make_workload, pack_bits_lsb  # noqa: E402


def goes_in_one_launch(ctx, call):
    """Whether the call was encode_few_kernel's: the other kernels quantise in a launch of their own or are counted."""
    ctx.hdc_profile_enable(True)
    call()
    n = {k: ctx.hdc_profile_read(k)[1] for k in ("encode", "quantize", "encode_contract", "encode_wide")}
    ctx.hdc_profile_enable(False)
    return n == dict(encode=1, quantize=0, encode_contract=0, encode_wide=0)


# on both sides of the lines: samples, blocks x (features + 160), blocks in the sparse encoder, planes of a count
@pytest.mark.parametrize("D,F,N,dense,sparse", [
    (500, 3, 1023, True, True), (500, 3, 1024, False, False), (10000, 561, 72, True, True), (10000, 561, 73, False, False),
    (10000, 3, 220, True, True), (10000, 3, 221, True, False), (10000, 3, 321, True, False), (10000, 3, 322, False, False),
    (1000, 4095, 2, True, True), (1000, 4096, 2, False, False)])
def test_which_calls_go_in_one_launch(D, F, N, dense, sparse):
    from paper_2206_04746_amd import binding
    wl = make_workload(2, seed=1, D=D, F=F, L=16, n_train=8)
    ctx = binding.Context(wl.D, wl.F, wl.L, wl.C, wl.item, wl.level, wl.tie, wl.lo, wl.scale, wl.dtype)
    x = torch.zeros((N, F), dtype=torch.float32, device="cuda")
    hv = torch.empty((N, ctx.W), dtype=torch.int32, device="cuda")
    assert goes_in_one_launch(ctx, lambda: ctx.hdc_encode(x, hv)) == dense
    assert goes_in_one_launch(ctx, lambda: ctx.hdc_encode_sparse(x, hv)) == sparse
    ctx.close()


@pytest.mark.parametrize("D,F,L,N,cfg", [
    (1, 1, 2, 1, 2), (33, 2, 3, 5, 2), (512, 31, 16, 3, 2), (513, 32, 64, 40, 2), (1000, 127, 100, 7, 2),
    (2048, 128, 256, 64, 2), (10000, 561, 100, 1, 2), (10000, 616, 64, 65, 2), (10016, 257, 64, 9, 2),
    (10000, 784, 256, 2, 3), (4000, 1024, 256, 12, 3), (1000, 4095, 16, 2, 2), (20000, 255, 1, 2, 2)])
@pytest.mark.parametrize("sparse", [False, True])
def test_few_samples_bit_exact(D, F, L, N, cfg, sparse):
    from paper_2206_04746_amd import binding
    wl = make_workload(cfg, seed=D + F, D=D, F=F, L=L, n_train=N)
    if N % 2:                                  # unrelated level vectors
        wl.level = pack_bits_lsb(np.random.default_rng(F).integers(0, 2, size=(L, D), dtype=np.uint8))
    x, _ = wl.train(N)
    if cfg == 2:
        x[0, 0], x[-1, -1] = np.nan, 2.0       # below and above the range
    ctx = binding.Context(wl.D, wl.F, wl.L, wl.C, wl.item, wl.level, wl.tie, wl.lo, wl.scale, wl.dtype)
    hv = torch.full((N, ctx.W), -1, dtype=torch.int32, device="cuda")
    (ctx.hdc_encode_sparse if sparse else ctx.hdc_encode)(torch.from_numpy(x).cuda(), hv)
    torch.cuda.synchronize()
    want = oracle.encode(x, wl.D, wl.L, wl.item, wl.level, wl.tie, wl.lo, wl.scale)
    assert np.array_equal(hv.cpu().numpy().view(np.uint32), want)
    ctx.close()
