"""The training kernel that holds B in registers (bf16, int8): bit-exact class
sums on integer inputs at the edges of its units, with rows that start at
every offset from a dword."""
from __future__ import annotations

import numpy as np
import pytest

import hd_inputs
import oracle
from gpu_util import announce, torch_or_skip

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hd():
    torch_or_skip()
    import paper_2506_09282_amd as m
    return m


def up(a, dtype, shift=0):
    torch = torch_or_skip()
    t = torch.from_numpy(np.ascontiguousarray(a)).cuda().to(
        torch.bfloat16 if dtype == "bf16" else torch.int8)
    buf = torch.zeros(t.numel() + shift, dtype=t.dtype, device="cuda")
    buf[shift:] = t.reshape(-1)
    return buf[shift:].view(t.shape)


def labels(N, K, seed):
    y = np.random.default_rng(seed).integers(-1, K + 1, N).astype(np.int32)  # some outside [0, K)
    if N > 4:
        y[:2] = (2 ** 30, -2 ** 30)
    return y


def run(hd, X, B, y, K, dtype, shift=0, counts=None):
    torch = torch_or_skip()
    c = hd.bundle_classes_packed(up(X, dtype, shift), hd.pack_model(up(B, dtype), K=K),
                                 torch.from_numpy(y).cuda(), K, counts=counts)
    torch.cuda.synchronize()
    return c.cpu().numpy()


# rows at one, two and four offsets from a dword; one f-step, a full and a
# ragged last one, the most for each count of class blocks (an int8 row of
# 1277 bytes takes 40 f-steps at every offset, one of 1279 does not fit);
# units of one sample, 31, 32, 33; the first and last class of a block
CASES = [("bf16", 1, 1, 100, 1), ("bf16", 31, 16, 64, 32), ("bf16", 33, 17, 300, 26),
         ("bf16", 64, 640, 256, 10), ("bf16", 65, 639, 257, 10), ("bf16", 500, 617, 1000, 26),
         ("bf16", 333, 511, 500, 33), ("bf16", 333, 512, 500, 64), ("bf16", 200, 319, 500, 65),
         ("bf16", 200, 320, 500, 128), ("bf16", 3, 3, 10240, 2),
         ("i8", 2, 1, 100, 3), ("i8", 130, 31, 300, 32), ("i8", 131, 33, 300, 26),
         ("i8", 132, 1280, 500, 5), ("i8", 133, 1277, 500, 5), ("i8", 133, 1279, 500, 5),
         ("i8", 700, 618, 1000, 26), ("i8", 701, 619, 1000, 60), ("i8", 300, 637, 300, 128)]


@pytest.mark.parametrize("dtype,N,F,D,K", CASES)
def test_integer_bit_exact(hd, dtype, N, F, D, K):
    announce(f"breg {dtype} N={N} F={F} D={D} K={K}")
    X, B, _ = hd_inputs.make_integer_inputs(N, F, D, 1, seed=N + F)
    y = labels(N, K, F)
    assert np.array_equal(run(hd, X, B, y, K, dtype), oracle.bundle(X, B, y, K)["counts"])


def test_many_units_per_workgroup(hd):
    """Several rounds of the LDS slots, with counts that are not zero before."""
    torch = torch_or_skip()
    N, F, D, K = 20001, 101, 10240, 9
    announce(f"breg N={N}")
    X, B, _ = hd_inputs.make_integer_inputs(N, F, D, 1, seed=8)
    y = labels(N, K, 8)
    c0 = torch.full((K, D), 5, dtype=torch.int32, device="cuda")
    assert np.array_equal(run(hd, X, B, y, K, "bf16", counts=c0),
                          oracle.bundle(X, B, y, K)["counts"] + 5)


@pytest.mark.parametrize("dtype,shift", [("bf16", 2), ("bf16", 1), ("i8", 4), ("i8", 3)])
def test_x_alignment(hd, dtype, shift):
    """X 4-byte aligned (this kernel) and not (X staged through registers)."""
    N, F, D, K = 99, 77, 300, 6
    announce(f"breg X shifted by {shift} {dtype}")
    X, B, _ = hd_inputs.make_integer_inputs(N, F, D, 1, seed=2)
    y = labels(N, K, 2)
    assert np.array_equal(run(hd, X, B, y, K, dtype, shift), oracle.bundle(X, B, y, K)["counts"])


@pytest.mark.parametrize("F", [36, 37])
def test_infinite_and_nan_features(hd, F):
    """A row's infinities and NaNs stay in the row."""
    N, D, K = 200, 256, 4
    announce(f"breg inf and nan F={F}")
    X, B, _ = hd_inputs.make_integer_inputs(N, F, D, 1, seed=6)
    B[5] = np.where(B[5] == 0, 1, B[5])
    X[3, 5], X[70, 5], X[120, F - 1], X[121, 0], X[60, F - 1] = np.inf, -np.inf, np.nan, np.nan, np.inf
    B[F - 1] = np.where(B[F - 1] == 0, 1, B[F - 1])
    y = labels(N, K, 6)
    assert np.array_equal(run(hd, X, B, y, K, "bf16"), oracle.bundle(X, B, y, K)["counts"])


@pytest.mark.parametrize("N,F,D", [(130, 51, 2048), (700, 617, 1000), (300, 5, 300), (300, 255, 512)])
def test_odd_rows_in_chunks(hd, N, F, D):
    """bf16 rows of odd length: the counts of one call bit for bit, from chunks
    that start at odd rows and from an X that starts inside a dword, on sums within
    rounding of zero (every row a multiple of one; the last three rows of B, at X = 1,
    cancel it to fp32's precision)."""
    torch = torch_or_skip()
    announce(f"breg odd rows in chunks N={N} F={F} D={D}")
    K, g = 4, np.random.default_rng(N + F)
    bf = lambda a: torch.from_numpy(a.astype(np.float32)).to(torch.bfloat16)
    x, B = bf(g.standard_normal(F)), bf(g.standard_normal((F, D)))
    x[-3:] = 1.0
    left = -(x[:-3].double() @ B[:-3].double())
    for i in range(3):
        B[F - 3 + i] = left.to(torch.bfloat16)
        left = left - B[F - 3 + i].double()
    X = (x.float() * torch.from_numpy(2.0 ** g.integers(-3, 4, (N, 1))).float()).to(torch.bfloat16)
    Xd = X.cuda()
    m = hd.pack_model(B.cuda(), K=K)
    yd = torch.from_numpy(g.integers(0, K, N).astype(np.int32)).cuda()
    one = hd.bundle_classes_packed(Xd, m, yd, K)
    for cuts in ((1, 60), (33, 34, 101), (N - 1,)):
        counts = torch.zeros_like(one)
        for a, b in zip((0,) + cuts, cuts + (N,)):
            hd.bundle_classes_packed(Xd[a:b], m, yd[a:b], K, counts=counts)
        torch.cuda.synchronize()
        assert torch.equal(one, counts), cuts
    buf = torch.zeros(N * F + 1, dtype=torch.bfloat16, device="cuda")
    buf[1:] = Xd.reshape(-1)
    shifted = hd.bundle_classes_packed(buf[1:].view(N, F), m, yd, K)
    torch.cuda.synchronize()
    assert torch.equal(one, shifted)
