"""The work that programs have this library do, as cases to be timed.

A case names an operation (a short sequence of entry points, as a program calls them), the model
(D dimensions, F features, L levels, C classes, element type of the features, kind of level table)
and the call (N samples, epochs, batch).  Sizes are those of this repository's workloads 1 to 6,
tests and benchmark; ``draw`` spreads them over the ranges in between.

Operations
  fit         encode the training set, add it up by class, binarise       (classical training)
  predict     encode the queries, nearest class by Hamming distance       (inference)
  step        fit, then search the same rows                              (one chunk of a long stream)
  search      nearest class of rows that are encoded already
  online      per-sample similarity-weighted training, binarise
  batched     the same with class rows frozen over a batch, binarise
  cosine      cosine inference against real-valued class rows
  primitives  pack, horizontal sum, vertical sum, unpack
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2206_04746_amd import binding

DEV = "cuda"


def _case(op, D, C, N, F=0, L=0, dtype="f32", levels="linear", encoder="dense", dist=False, epochs=1, batch=0):
    return dict(op=op, D=D, F=F, L=L, C=C, N=N, dtype=dtype, levels=levels, encoder=encoder, dist=dist,
                epochs=epochs, batch=batch)


def listed():
    return [
        # one window at a time, as a wearable or a request handler classifies it: launches and latency
        dict(_case("predict", D=10000, F=561, L=100, C=6, N=1), name="predict-one"),
        # the test set of the spoken-letter shape (workload 2), distances kept for a confidence
        dict(_case("predict", D=10000, F=617, L=64, C=26, N=1559, dist=True), name="predict-isolet"),
        # small F, ordinary size: the activity-monitoring shape (workload 6), inference
        dict(_case("predict", D=10000, F=31, L=64, C=5, N=16000), name="predict-pamap"),
        # the tiny model (workload 1): training where launches count
        dict(_case("fit", D=1024, F=100, L=16, C=5, N=2000), name="fit-tiny"),
        # the training set of workload 2
        dict(_case("fit", D=10000, F=617, L=64, C=26, N=6238), name="fit-isolet"),
        # digit images (workload 3): bytes, four fifths zero, level vectors without structure, the
        # encoder for inputs that mostly sit in the lowest bin
        dict(_case("fit", D=10000, F=784, L=256, C=10, N=60000, dtype="u8", levels="random", encoder="sparse"),
             name="fit-digits-sparse"),
        # a chunk of the long EEG stream (workload 5, the benchmark's step): the largest
        dict(_case("step", D=10000, F=342, L=64, C=2, N=1000000), name="step-eeg"),
        # a long stream of encoded rows against many classes, distances wanted
        dict(_case("search", D=10000, C=26, N=1000000, dist=True), name="search-stream"),
        # per-sample online training at workload 4: three passes over 7352 windows
        dict(_case("online", D=10000, F=561, L=100, C=6, N=7352, epochs=3), name="online-ucihar"),
        # the same set, class rows updated after every 64 windows
        dict(_case("batched", D=10000, F=561, L=100, C=6, N=7352, batch=64), name="batched-ucihar"),
        # its test set by cosine against the real-valued rows
        dict(_case("cosine", D=10000, F=561, L=100, C=6, N=2947), name="cosine-ucihar"),
        # the stand-alone primitives on one large matrix of bits
        dict(_case("primitives", D=10000, C=2, N=131072), name="primitives"),
    ]


def _log(rng, lo, hi):
    """A whole number spread evenly over the logarithm of [lo, hi]."""
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _model(rng):
    """F, L, dtype, levels, encoder of a drawn model.  Most level tables step linearly between two
    vectors; circles (periodic quantities) and unstructured tables are the other kinds in use."""
    sparse = rng.random() < 0.2
    return dict(F=_log(rng, 24, 800), L=rng.choice([16, 32, 50, 64, 100, 128, 200, 256]),
                dtype="u8" if sparse or rng.random() < 0.2 else "f32",
                levels=rng.choice(["linear", "linear", "linear", "linear", "circular", "random"]),
                encoder="sparse" if sparse else "dense")


def draw(rng):
    op = rng.choice(["fit", "predict", "predict", "step", "search", "online", "batched", "cosine", "primitives"])
    if op == "fit":
        return _case(op, D=_log(rng, 1000, 20000), C=_log(rng, 2, 64), N=_log(rng, 500, 65536), **_model(rng))
    if op == "predict":
        return _case(op, D=_log(rng, 1000, 20000), C=_log(rng, 2, 64), N=_log(rng, 1, 65536),
                     dist=rng.random() < 0.5, **_model(rng))
    if op == "step":   # long streams: 24 to 400 features, few classes
        D, F = _log(rng, 4000, 16384), _log(rng, 24, 400)
        most = min(1000000, int(2.5e9 / (4 * F + D / 8)), int(3.0e12 / (F * D)))
        return _case(op, D=D, C=rng.choice([2, 2, 3, 5, 8]), N=_log(rng, most // 8, most), F=F, L=rng.choice([32, 64]))
    if op == "search":
        D, C = _log(rng, 1000, 32768), _log(rng, 2, 200)
        return _case(op, D=D, C=C, N=_log(rng, 100, min(1000000, int(1.0e10 / D), int(8e11 / (C * D)))),
                     dist=rng.random() < 0.5)
    if op == "primitives":
        D = _log(rng, 1000, 32768)
        return _case(op, D=D, C=2, N=_log(rng, 500, int(1.3e9 / D)))
    # the online family: encoded sets of a few thousand samples
    base = dict(D=_log(rng, 1000, 12000), C=_log(rng, 2, 26), F=_log(rng, 24, 600), L=rng.choice([16, 64, 100]))
    if op == "online":
        return _case(op, N=_log(rng, 300, 5000), epochs=rng.choice([1, 1, 2]), **base)
    if op == "batched":
        n = _log(rng, 500, 8000)
        return _case(op, N=n, batch=_log(rng, 8, min(n, 4096)), **base)
    return _case(op, N=_log(rng, 1, 20000), **base)


# ------------------------------------------------------------------------------------- inputs
def _words(rng, rows, D):
    """Random hypervectors, packed: [rows][W] uint32, pad bits zero."""
    W = (D + 31) // 32
    t = rng.integers(0, 1 << 32, size=(rows, W), dtype=np.uint32)
    if D % 32:
        t[:, -1] &= np.uint32((1 << (D % 32)) - 1)
    return t


def _pack(bits):
    L, D = bits.shape
    out = np.zeros((L, (D + 31) // 32 * 32), dtype=np.uint8)
    out[:, :D] = bits
    return np.ascontiguousarray(np.packbits(out, axis=1, bitorder="little")).view("<u4")


def _level_table(rng, D, L, kind):
    """linear: every step flips fresh dimensions, half of them in all.  circular: the second half of
    the circle flips them back.  random: independent vectors."""
    if kind == "random":
        return _words(rng, L, D)
    steps = L - 1 if kind == "linear" else L // 2
    b = D // (2 * steps)
    perm = rng.permutation(D)
    bits = np.empty((L, D), dtype=np.uint8)
    bits[0] = rng.integers(0, 2, size=D, dtype=np.uint8)
    for k in range(1, L):
        j = (k - 1) % steps
        bits[k] = bits[k - 1]
        bits[k, perm[j * b:(j + 1) * b]] ^= 1
    return _pack(bits)


def _features(case, g):
    """Feature rows and labels on the GPU: clusters clipped to [-1, 1] (workloads 2, 4, 6), bytes with
    a mostly dark background (workload 3), or log-normal rows of which one in a hundred, in runs, is
    positive (workload 5)."""
    N, F, C = case["N"], case["F"], case["C"]
    if case["op"] == "step":
        run = torch.rand((N + 63) // 64, device=DEV, generator=g) < (0.01 if C == 2 else 0.5)
        y = run.to(torch.int32).repeat_interleave(64)[:N].contiguous()
        if C > 2:
            y = y * torch.randint(1, C, (N,), device=DEV, generator=g, dtype=torch.int32)
        mu = torch.rand(F, device=DEV, generator=g) - 0.5
        x = torch.randn((N, F), device=DEV, generator=g).mul_(0.5).add_(mu).add_(0.5 / (C - 1) * y[:, None]).exp_()
        return x, y, np.zeros(F), np.exp(mu.cpu().numpy().astype(np.float64) + 3.0902 * 0.5)
    y = torch.randint(0, C, (N,), device=DEV, generator=g, dtype=torch.int32)
    if case["dtype"] == "u8":
        on = torch.rand((C, F), device=DEV, generator=g) < 0.2
        keep = torch.rand((N, F), device=DEV, generator=g) < torch.where(on, 0.9, 0.01)[y.long()]
        x = torch.randint(64, 256, (N, F), device=DEV, generator=g, dtype=torch.int32).mul_(keep).to(torch.uint8)
        return x, y, None, None
    means = torch.rand((C, F), device=DEV, generator=g) - 0.5
    x = means[y.long()] + 0.25 * torch.randn((N, F), device=DEV, generator=g)
    return x.clamp_(-1.0, 1.0), y, -np.ones(F), np.ones(F)


def _rows(case, g):
    """Encoded rows and class vectors as a trained model sees them: a class's rows differ from its
    vector in about a quarter of the dimensions."""
    D, W, N, C = case["D"], (case["D"] + 31) // 32, case["N"], case["C"]

    def words(n):
        return torch.randint(-(1 << 31), 1 << 31, (n, W), device=DEV, generator=g, dtype=torch.int32)

    cls = words(C)
    y = torch.randint(0, C, (N,), device=DEV, generator=g, dtype=torch.int32)
    hv = words(N).bitwise_and_(words(N)).bitwise_xor_(cls[y.long()])
    if D % 32:
        last = (1 << (D % 32)) - 1
        cls[:, -1] &= last
        hv[:, -1] &= last
    return hv, y, cls


def prepare(case, seed):
    op, D, N, C = case["op"], case["D"], case["N"], case["C"]
    W = (D + 31) // 32
    rng = np.random.default_rng([seed, D, N])
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    new = lambda shape, dtype=torch.int32: torch.zeros(shape, dtype=dtype, device=DEV)  # noqa: E731
    s = dict(case=case)
    if op in ("search", "primitives"):
        # no encoding: a model of one feature carries D and C
        s["ctx"] = binding.Context(D, 1, 2, C, _words(rng, 1, D), _words(rng, 2, D), _words(rng, 1, D)[0], None, None, "u8")
        if op == "primitives":
            s["bits"] = torch.randint(0, 2, (N, D), device=DEV, generator=g, dtype=torch.uint8)
            s.update(hv=new((N, W)), hsum=new(N), vsum=new(D), back=new((N, D), torch.uint8))
        else:
            s["hv"], _, s["cls"] = _rows(case, g)
            s.update(pred=new(N), dist=new((N, C)) if case["dist"] else None)
        return s
    F, L = case["F"], case["L"]
    item, level, tie = _words(rng, F, D), _level_table(rng, D, L, case["levels"]), _words(rng, 1, D)[0]
    x, y, lo, hi = _features(case, g)
    scale = None if lo is None else (L / (hi - lo)).astype(np.float32)
    ctx = binding.Context(D, F, L, C, item, level, tie, lo, scale, case["dtype"])
    s.update(ctx=ctx, x=x, y=y, hv=new((N, W)), cls=new((C, W)))
    if case["encoder"] == "sparse":
        ctx.hdc_reserve(binding.HDC_RESERVE_ENCODE_SPARSE)
    if op in ("fit", "step"):
        s.update(acc=new((C, D)), cn=new(C, torch.int64))
    if op == "predict":
        s["cls"] = torch.from_numpy(_words(rng, C, D).view(np.int32)).to(DEV)
    if op in ("predict", "step"):
        s.update(pred=new(N), dist=new((N, C)) if case["dist"] else None)
    if op in ("online", "batched", "cosine"):
        # the set is encoded once and trained on, or searched, from there
        ctx.hdc_encode(x, s["hv"])
        s["acc"] = new((C, D), torch.float32)
        if op == "online":
            ctx.hdc_reserve(binding.HDC_RESERVE_ONLINE)
        if op == "batched":
            ctx.hdc_reserve(binding.HDC_RESERVE_ONLINE_BATCHED, max_batch=case["batch"])
        if op == "cosine":
            ctx.hdc_reserve(binding.HDC_RESERVE_SEARCH_COSINE, max_queries=N)
            # rows as training leaves them: the sums of a few hundred weighted samples
            s["acc"].copy_(torch.randn((C, D), device=DEV, generator=g).mul_(12.0))
            s.update(pred=new(N), cos=new((N, C), torch.float32))
    return s


def _encode(s):
    (s["ctx"].hdc_encode_sparse if s["case"]["encoder"] == "sparse" else s["ctx"].hdc_encode)(s["x"], s["hv"])


def run(s):
    case, ctx = s["case"], s["ctx"]
    op = case["op"]
    if op == "predict":
        _encode(s)
        ctx.hdc_search(s["hv"], s["cls"], s["pred"], s["dist"])
        return s["hv"], s["pred"], s["dist"]
    if op in ("fit", "step"):
        s["acc"].zero_()
        s["cn"].zero_()
        _encode(s)
        ctx.hdc_train_classical(s["hv"], s["y"], s["acc"], s["cn"])
        ctx.hdc_binarize_classical(s["acc"], s["cn"], s["cls"])
        if op == "fit":
            return s["hv"], s["acc"], s["cn"], s["cls"]
        ctx.hdc_search(s["hv"], s["cls"], s["pred"], s["dist"])
        return s["hv"], s["acc"], s["cn"], s["cls"], s["pred"]
    if op == "search":
        ctx.hdc_search(s["hv"], s["cls"], s["pred"], s["dist"])
        return s["pred"], s["dist"]
    if op in ("online", "batched"):
        s["acc"].zero_()
        if op == "online":
            ctx.hdc_train_online(s["hv"], s["y"], s["acc"], epochs=case["epochs"], lr=1.0)
        else:
            ctx.hdc_train_online_batched(s["hv"], s["y"], s["acc"], batch=case["batch"], epochs=case["epochs"], lr=1.0)
        ctx.hdc_binarize_online(s["acc"], s["cls"])
        return s["acc"], s["cls"]
    if op == "cosine":
        ctx.hdc_search_cosine(s["hv"], s["acc"], s["pred"], s["cos"])
        return s["pred"], s["cos"]
    ctx.hdc_pack(s["bits"], s["hv"])
    ctx.hdc_hsum(s["hv"], s["hsum"])
    ctx.hdc_vsum(s["hv"], s["vsum"])
    ctx.hdc_unpack(s["hv"], s["back"])
    return s["hv"], s["hsum"], s["vsum"], s["back"]


def work(case):
    """Inputs read once, outputs written once.  Operations: an add per (feature, dimension) for
    encoding, where a dimension on which all level vectors agree is a constant and costs nothing, an
    add per (row, dimension) for sums, a multiply and an add per (row, class, dimension) for
    distances and cosines."""
    op, D, F, N, C = case["op"], case["D"], case["F"], case["N"], case["C"]
    row, esz = (D + 31) // 32 * 4, 1 if case["dtype"] == "u8" else 4
    moving = D
    if F and case["levels"] != "random":
        steps = case["L"] - 1 if case["levels"] == "linear" else case["L"] // 2
        moving = D // (2 * steps) * steps
    model = (F + case["L"] + 1) * row
    found = N * 4 + (N * C * 4 if case["dist"] else 0)
    if op == "predict":
        return dict(bytes=N * (F * esz + row) + model + C * row + found, flops=N * (F * moving + 2 * C * D))
    if op in ("fit", "step"):
        b = N * (F * esz + row + 4) + model + C * (4 * D + 8 + row)
        f = N * (F * moving + D)
        return dict(bytes=b + (found if op == "step" else 0), flops=f + (2 * N * C * D if op == "step" else 0))
    if op == "search":
        return dict(bytes=N * row + C * row + found, flops=2 * N * C * D)
    if op in ("online", "batched"):
        return dict(bytes=N * (row + 4) + C * (4 * D + row), flops=case["epochs"] * N * (2 * C * D + 4 * D))
    if op == "cosine":
        return dict(bytes=N * row + 4 * C * D + N * 4 * (1 + C), flops=2 * N * C * D)
    return dict(bytes=2 * N * D + N * row + 4 * N + 4 * D, flops=2 * N * D)


def tolerance(case):
    """Integer work is exact.  Online rows are fp32 sums of fp32 weights that come from fp64 cosines:
    another order of summation moves a weight by a last bit now and then, and the sign of an element
    next to zero with it.  Cosines are fp64 sums rounded once; two classes may tie to the last bit."""
    if case["op"] in ("online", "batched"):
        return {"rel": 1e-5, "max": 1e-3, "differ": 2e-3}
    if case["op"] == "cosine":
        return {"rel": 1e-6, "max": 1e-5, "differ": 1e-3}
    return "exact"
