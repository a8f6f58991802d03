"""Boundary behaviour that is not arithmetic (the calls the C ABI lists beside the operations of
the paper): label checking (labels outside [0, C) are skipped by default and refused with
HDC_ELABEL when checking is on, Sec. III's training calls), and hdc_reserve (after it, the calls
that otherwise allocate at first use give the same results and allocate nothing more)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
from workloads import make_workload  # noqa: E402


def _setup(n=600):
    from paper_2206_04746_amd import binding
    wl = make_workload(1, n_train=n)
    x, y = wl.train(n)
    ctx = binding.Context(wl.D, wl.F, wl.L, wl.C, wl.item, wl.level, wl.tie, wl.lo, wl.scale, wl.dtype)
    hv = torch.empty((n, ctx.W), dtype=torch.int32, device="cuda")
    ctx.hdc_encode(torch.from_numpy(x).cuda(), hv)
    return binding, wl, ctx, hv, y


def test_label_check_refuses_out_of_range_labels_and_trains_nothing():
    binding, wl, ctx, hv, y = _setup()
    bad = y.copy()
    bad[17] = wl.C
    bad[400] = -1
    yd, bd = torch.from_numpy(y).cuda(), torch.from_numpy(bad).cuda()
    acc = torch.zeros((wl.C, wl.D), dtype=torch.int32, device="cuda")
    cn = torch.zeros(wl.C, dtype=torch.int64, device="cuda")
    facc = torch.zeros((wl.C, wl.D), dtype=torch.float32, device="cuda")
    # default: such samples are skipped
    ctx.hdc_train_classical(hv, bd, acc, cn)
    torch.cuda.synchronize()
    hv_h = hv.cpu().numpy().view(np.uint32)
    o_acc, o_cn = oracle.train_classical(hv_h, bad, wl.D, wl.C)
    assert np.array_equal(acc.cpu().numpy(), o_acc) and int(cn.sum()) == len(y) - 2
    # checking on: refused, nothing touched
    ctx.hdc_set_label_check(True)
    acc.zero_(), cn.zero_()
    for call in (lambda: ctx.hdc_train_classical(hv, bd, acc, cn),
                 lambda: ctx.hdc_train_online(hv, bd, facc, 1, 1.0),
                 lambda: ctx.hdc_train_online_batched(hv, bd, facc, 64, 1, 1.0)):
        with pytest.raises(binding.HdcError) as err:
            call()
        assert err.value.code == binding.HDC_ELABEL
    torch.cuda.synchronize()
    assert int(acc.abs().sum()) == 0 and int(cn.sum()) == 0 and float(facc.abs().sum()) == 0.0
    assert "label" in binding.strerror(binding.HDC_ELABEL)
    # good labels pass with checking on, and give the usual result
    ctx.hdc_train_classical(hv, yd, acc, cn)
    torch.cuda.synchronize()
    o_acc, o_cn = oracle.train_classical(hv_h, y, wl.D, wl.C)
    assert np.array_equal(acc.cpu().numpy(), o_acc) and np.array_equal(cn.cpu().numpy(), o_cn)
    ctx.hdc_set_label_check(False)
    ctx.close()


def test_reserve_then_calls_allocate_nothing_and_match():
    binding, wl, ctx, hv, y = _setup()
    yd = torch.from_numpy(y).cuda()
    n = hv.shape[0]
    ctx.hdc_reserve(binding.HDC_RESERVE_ONLINE | binding.HDC_RESERVE_ONLINE_BATCHED | binding.HDC_RESERVE_SEARCH_COSINE
                    | binding.HDC_RESERVE_ENCODE_SPARSE, max_batch=256, max_queries=n)
    torch.cuda.synchronize()
    facc = torch.zeros((wl.C, wl.D), dtype=torch.float32, device="cuda")
    facb = torch.zeros((wl.C, wl.D), dtype=torch.float32, device="cuda")
    pred = torch.empty(n, dtype=torch.int32, device="cuda")
    cos = torch.empty((n, wl.C), dtype=torch.float32, device="cuda")
    x, _ = wl.train(n)
    hv2 = torch.empty_like(hv)
    xd = torch.from_numpy(x).cuda()
    free0 = torch.cuda.mem_get_info()[0]
    ctx.hdc_train_online(hv, yd, facc, 2, 1.0)
    ctx.hdc_train_online_batched(hv, yd, facb, 256, 2, 1.0)
    ctx.hdc_search_cosine(hv, facb, pred, cos)
    ctx.hdc_encode_sparse(xd, hv2)
    torch.cuda.synchronize()
    # (the HIP runtime may take a few MB of its own at a kernel's first launch; the scratch these calls would
    # allocate without hdc_reserve is 12.7 MB for hdc_train_online alone)
    assert free0 - torch.cuda.mem_get_info()[0] < (8 << 20), "a call after hdc_reserve allocated device memory"
    hv_h = hv.cpu().numpy().view(np.uint32)
    want = oracle.train_online(hv_h, y, wl.D, wl.C, epochs=2, lr=1.0)
    assert np.max(np.abs(facc.cpu().numpy() - want) / np.maximum(np.abs(want), 1e-3 * np.abs(want).max())) < 1e-4
    wantb = oracle.train_online_batched(hv_h, y, wl.D, wl.C, 256, 2, 1.0)
    assert np.max(np.abs(facb.cpu().numpy() - wantb)) <= 1e-5 * np.abs(wantb).max()
    o_cos, _ = oracle.search_cosine(hv_h, facb.cpu().numpy(), wl.D)
    assert float(np.max(np.abs(cos.cpu().numpy() - o_cos))) <= 1e-5
    assert torch.equal(hv2, hv)
    # bad arguments
    with pytest.raises(binding.HdcError) as err:
        ctx.hdc_reserve(binding.HDC_RESERVE_ONLINE_BATCHED, max_batch=0)
    assert err.value.code == binding.HDC_EINVAL
    with pytest.raises(binding.HdcError):
        ctx.hdc_reserve(1 << 9)
    ctx.close()


def test_reserved_calls_are_captured_without_a_call_before():
    """Nothing may be allocated under capture, so this fails for whatever hdc_reserve left out."""
    binding, wl, ctx, hv, y = _setup()
    yd = torch.from_numpy(y).cuda()
    n = hv.shape[0]
    ctx.hdc_reserve(binding.HDC_RESERVE_ONLINE | binding.HDC_RESERVE_ONLINE_BATCHED | binding.HDC_RESERVE_SEARCH_COSINE
                    | binding.HDC_RESERVE_ENCODE_SPARSE, max_batch=256, max_queries=n)
    rows = [torch.empty((wl.C, wl.D), dtype=torch.float32, device="cuda") for _ in range(4)]
    pred = torch.empty(n, dtype=torch.int32, device="cuda")
    x, _ = wl.train(n)
    xd = torch.from_numpy(x).cuda().repeat(8, 1)               # (more than a few samples)
    hv2 = torch.empty((8 * n, ctx.W), dtype=torch.int32, device="cuda")
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        for r in rows:
            r.zero_()
        ctx.hdc_train_online(hv, yd, rows[0], 2, 1.0)
        ctx.hdc_train_online(hv[:3], yd[:3], rows[1], 1, 1.0)
        ctx.hdc_train_online_batched(hv, yd, rows[2], 256, 2, 1.0)
        ctx.hdc_train_online_batched(hv, yd, rows[3], 16, 2, 1.0)
        ctx.hdc_search_cosine(hv, rows[2], pred, None)
        ctx.hdc_encode_sparse(xd, hv2)
    hv_h = hv.cpu().numpy().view(np.uint32)
    want = [oracle.train_online(hv_h, y, wl.D, wl.C, 2, 1.0), oracle.train_online(hv_h[:3], y[:3], wl.D, wl.C, 1, 1.0),
            oracle.train_online_batched(hv_h, y, wl.D, wl.C, 256, 2, 1.0), oracle.train_online_batched(hv_h, y, wl.D, wl.C, 16, 2, 1.0)]
    for _ in range(3):
        graph.replay()
        torch.cuda.synchronize()
        for got, w in zip(rows, want):
            assert np.max(np.abs(got.cpu().numpy() - w)) <= 1e-5 * np.abs(w).max()
        o_cos, o_pred = oracle.search_cosine(hv_h, rows[2].cpu().numpy(), wl.D)
        assert np.array_equal(pred.cpu().numpy(), o_pred)
        assert torch.equal(hv2, hv.repeat(8, 1))
        for r in rows:
            r.fill_(3.0)
    ctx.close()


def test_search_of_one_chunk_beside_the_encoding_of_the_next_on_two_streams():
    """hdc_search uses no scratch of the context, so with one context the search of chunk k may run
    on one stream while chunk k + 1 is encoded on another (a long stream invites
    that): the rows and predictions equal those of the same calls made one after the other."""
    wl = make_workload(5)
    from paper_2206_04746_amd import binding
    n = 65000                                    # per chunk: enough for the long-stream encoder
    x, y = wl.train(3 * n)
    ctx = binding.Context(wl.D, wl.F, wl.L, wl.C, wl.item, wl.level, wl.tie, wl.lo, wl.scale, wl.dtype)
    xd = torch.from_numpy(x).cuda()
    yd = torch.from_numpy(y.astype(np.int32)).cuda()
    hv_ref = torch.empty((3 * n, ctx.W), dtype=torch.int32, device="cuda")
    ctx.hdc_encode(xd, hv_ref)
    acc = torch.zeros((wl.C, wl.D), dtype=torch.int32, device="cuda")
    cn = torch.zeros(wl.C, dtype=torch.int64, device="cuda")
    ctx.hdc_train_classical(hv_ref, yd, acc, cn)
    cls = torch.empty((wl.C, ctx.W), dtype=torch.int32, device="cuda")
    ctx.hdc_binarize_classical(acc, cn, cls)
    pred_ref = torch.empty(3 * n, dtype=torch.int32, device="cuda")
    ctx.hdc_search(hv_ref, cls, pred_ref, None)
    torch.cuda.synchronize()

    hv = torch.full((3 * n, ctx.W), -1, dtype=torch.int32, device="cuda")
    pred = torch.full((3 * n,), -1, dtype=torch.int32, device="cuda")
    torch.cuda.synchronize()
    s_enc, s_srch = torch.cuda.Stream(), torch.cuda.Stream()
    done = [torch.cuda.Event() for _ in range(3)]
    for k in range(3):
        with torch.cuda.stream(s_enc):
            ctx.hdc_encode(xd[k * n:(k + 1) * n], hv[k * n:(k + 1) * n])
            done[k].record(s_enc)
        with torch.cuda.stream(s_srch):
            s_srch.wait_event(done[k])           # chunk k is searched once it is encoded, beside the encoding of k + 1
            ctx.hdc_search(hv[k * n:(k + 1) * n], cls, pred[k * n:(k + 1) * n], None)
    torch.cuda.synchronize()
    assert torch.equal(hv, hv_ref)
    assert torch.equal(pred, pred_ref)
    ctx.close()
