"""The workloads this library's speed is measured on: plain cases, each run
through the package's public entry points.

Shapes follow ``hd_inputs.WORKLOADS`` (F, K and the distribution of X), the
dimension D = 10240 of the benchmark and the paper's own D = 10000. A case
names its call:

* ``infer_packed``: Alg. 1 on a model tiled once, the serving path;
* ``infer``: Alg. 1 on B and C as given (one-off calls, models that change);
* ``infer_stream``: one launch over a queue of small batches;
* ``train_packed``: one chunk of single-pass training, the class sums (the
  state that the chunks accumulate; the codebook is their sign, taken once);
* ``bundle``: the same on B as given.
"""
from __future__ import annotations

import math

import torch

import paper_2506_09282_amd as hd

DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16, "i8": torch.int8}
ESIZE = {"f32": 4, "bf16": 2, "i8": 1}

# Rough device rates (multiply-adds counted as two), only to keep drawn cases
# below the largest listed one.
RATE = {"f32": 60e12, "bf16": 350e12, "i8": 600e12}
MOST_SECONDS = 3e-3
MOST_FLOPS = 9e11


def _case(name, call, dtype, N, F, D, K, x, nbatch=1, det=False):
    c = {"call": call, "dtype": dtype, "N": N, "F": F, "D": D, "K": K, "x": x, "nbatch": nbatch,
         "det": det}
    return {"name": name, **c} if name else c


def listed():
    return [
        # one reading of a wearable sensor, answered as it arrives (latency)
        _case("activity_n1_f32", "infer_packed", "f32", 1, 561, 10240, 6, "pm1"),
        # a small request batch of the same service: the benchmark's default
        _case("activity_n32_f32", "infer_packed", "f32", 32, 561, 10240, 6, "pm1"),
        # a middling request batch on a bf16 model, not a multiple of any tile
        _case("activity_n100_bf16", "infer_packed", "bf16", 100, 561, 10240, 6, "pm1"),
        # a test-set chunk of 28x28 images on a bf16 model
        _case("image_bf16", "infer_packed", "bf16", 4096, 784, 10240, 10, "u01z"),
        # the same in fp32, the precision the paper keeps
        _case("image_f32", "infer_packed", "f32", 4096, 784, 10240, 10, "u01z"),
        # bulk classification of spoken letters; rows of odd length
        _case("speech_bf16", "infer_packed", "bf16", 65536, 617, 10240, 26, "normal"),
        # the same on a quantised model
        _case("speech_i8", "infer_packed", "i8", 65536, 617, 10240, 26, "i8"),
        # bulk classification of 32x32x3 images: wide features
        _case("colour_bf16", "infer_packed", "bf16", 16384, 3072, 10240, 10, "u01"),
        # one-off evaluation of matrices as given, at the paper's D
        _case("speech_raw_f32", "infer", "f32", 500, 617, 10000, 26, "normal"),
        # a real-time queue of small batches in one launch
        _case("activity_stream_f32", "infer_stream", "f32", 32, 561, 10240, 6, "pm1", nbatch=256),
        # single-pass training on a bulk set; rows of odd length
        _case("speech_train_bf16", "train_packed", "bf16", 65536, 617, 10240, 26, "normal"),
        # one chunk of a training set, on base vectors as given
        _case("image_bundle_f32", "bundle", "f32", 2048, 784, 10240, 10, "u01z"),
    ]


def _log(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    call = rng.choice(["infer_packed"] * 6 + ["infer", "infer_stream", "train_packed", "bundle"])
    dtype = rng.choice(["f32", "bf16", "i8"])
    x = rng.choice(["pm1", "u01", "u01z", "normal"])
    D = rng.choice([10240, 10000, rng.randint(1000, 12240)])
    if call == "infer_stream":
        return _case(None, call, "f32", _log(rng, 1, 32), _log(rng, 32, 576), D, rng.randint(2, 16),
                     x, nbatch=_log(rng, 16, 256))
    if call == "bundle" and dtype == "i8":  # B as given: fp32 and bf16 only
        dtype = "bf16"
    F, K, N = _log(rng, 32, 3072), _log(rng, 2, 100), _log(rng, 1, 65536)
    if call in ("train_packed", "bundle"):
        N = max(N, 256)
    rate = RATE[dtype] / (2 if call in ("train_packed", "infer") else 4 if call == "bundle" else 1)
    if call == "bundle":
        rate = min(rate, 30e12)
    per = 2.0 * D * (F + K)
    N = max(1, min(N, int(MOST_FLOPS / per), int(MOST_SECONDS * rate / per)))
    det = call in ("infer_packed", "infer") and rng.random() < 0.2
    return _case(None, call, dtype, N, F, D, K, "i8" if dtype == "i8" else x, det=det)


def _inputs(case, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    n, F, D, K = case["N"] * case["nbatch"], case["F"], case["D"], case["K"]
    if case["dtype"] == "i8":
        def ints(*shape):
            return torch.randint(-128, 128, shape, dtype=torch.int8, device="cuda", generator=g)
        return ints(n, F), ints(F, D), ints(K, D), g
    kind, dt = case["x"], DTYPES[case["dtype"]]
    if kind == "normal":
        X = torch.randn(n, F, device="cuda", generator=g)
    else:
        X = torch.rand(n, F, device="cuda", generator=g)
        if kind == "pm1":
            X = X * 2 - 1
        elif kind == "u01z":  # dark pixels
            X = X * (torch.rand(n, F, device="cuda", generator=g) >= 0.2)
    B = torch.randn(F, D, device="cuda", generator=g)
    C = torch.randn(K, D, device="cuda", generator=g)
    return X.to(dt), B.to(dt), C.to(dt), g


def _labels(case, g):
    return torch.randint(0, case["K"], (case["N"],), dtype=torch.int32, device="cuda", generator=g)


def prepare(case, seed):
    X, B, C, g = _inputs(case, seed)
    N, F, D, K, dt = case["N"], case["F"], case["D"], case["K"], X.dtype
    s = {"call": case["call"], "K": K, "det": case["det"], "X": X}
    if case["call"] == "train_packed":
        s["y"], s["model"] = _labels(case, g), hd.pack_model(B, K=K)
    elif case["call"] == "bundle":
        s["y"], s["B"] = _labels(case, g), B
    elif case["call"] == "infer":
        s["B"], s["C"] = B, C
    else:
        s["model"] = hd.pack_model(B, C)
        if case["call"] == "infer_stream":
            s["X"] = X.view(case["nbatch"], N, F)
            need = hd.stream_workspace_bytes(case["nbatch"], N, F, D, K, dt)
            s["out"] = (torch.empty((case["nbatch"], N), dtype=torch.int32, device="cuda"),
                        torch.empty((case["nbatch"], N, K), dtype=torch.float32, device="cuda"))
            s["ws"] = torch.zeros(need, dtype=torch.uint8, device="cuda")
        elif N <= 256:  # a serving loop keeps its outputs
            s["out"] = (torch.empty(N, dtype=torch.int32, device="cuda"),
                        torch.empty((N, K), dtype=torch.float32, device="cuda"))
    return s


def run(s):
    call = s["call"]
    if call == "infer_packed":
        return hd.infer_packed(s["X"], s["model"], return_scores=True, out=s.get("out"),
                               deterministic=s["det"])
    if call == "infer":
        return hd.infer(s["X"], s["B"], s["C"], return_scores=True, deterministic=s["det"])
    if call == "infer_stream":
        return hd.infer_stream(s["X"], s["model"], return_scores=True, out=s["out"],
                               workspace=s["ws"])
    if call == "train_packed":
        return hd.bundle_classes_packed(s["X"], s["model"], s["y"], s["K"])
    return hd.bundle_classes(s["X"], s["B"], s["y"], s["K"])


def work(case):
    """X, B (and C or the labels) read once, the results written once; two
    operations per multiply-add of Stage I and, in inference, Stage II."""
    n, F, D, K, e = case["N"] * case["nbatch"], case["F"], case["D"], case["K"], ESIZE[case["dtype"]]
    if case["call"] in ("train_packed", "bundle"):
        return {"bytes": e * (n * F + F * D) + 4 * n + 4 * K * D, "flops": 2 * n * D * F}
    return {"bytes": e * (n * F + F * D + K * D) + 4 * n + 4 * n * K, "flops": 2 * n * D * (F + K)}


def tolerance(case):
    """int8 is exact. Elsewhere HardSign is taken on an fp32 sum of F products,
    so a dimension whose product lies within that sum's rounding of zero can
    take either sign: measured below 1e-6 of the dimensions. One such
    dimension moves a row's scores by 2 |c| against sqrt(D) |c|."""
    if case["dtype"] == "i8":
        return "exact"
    n, D = case["N"] * case["nbatch"], case["D"]
    flips = 2.0 + 2e-6 * n * D
    if case["call"] in ("train_packed", "bundle"):
        # each flip moves one class sum by 2
        return {"rel": 0.02, "max": 0.9, "differ": min(0.01, flips / (case["K"] * D))}
    return {"rel": min(0.03, max(1e-5, 2.0 * math.sqrt(flips / (n * D)))), "max": 0.9,
            "differ": 2e-3}


def exact(case, seed):
    X, B, C, g = _inputs(case, seed)
    n, D, K = X.shape[0], case["D"], case["K"]
    Bd, Cd = B.double(), C.double()
    train = case["call"] in ("train_packed", "bundle")
    y = _labels(case, g).long() if train else None
    counts = torch.zeros(K, D, dtype=torch.float64, device="cuda")
    scores = torch.empty(n, K, dtype=torch.float64, device="cuda")
    for r0 in range(0, n, 4096):
        V = X[r0:r0 + 4096].double() @ Bd
        H = torch.where(V >= 0, 1.0, -1.0).double()
        if train:
            hot = torch.nn.functional.one_hot(y[r0:r0 + 4096], K).double()
            counts += hot.t().contiguous() @ H
        else:
            scores[r0:r0 + 4096] = H @ Cd.t().contiguous()
    if train:
        return counts.to(torch.int32)
    labels = scores.argmax(dim=1).to(torch.int32)
    if case["call"] == "infer_stream":
        shape = (case["nbatch"], case["N"])
        return labels.view(shape), scores.view(*shape, K)
    return labels, scores
