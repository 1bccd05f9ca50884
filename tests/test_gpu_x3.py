"""fp32 Stage I on the bf16 matrix instruction (large batches, training; B packed
and as given): bit-exact on integer inputs at the edges of its tiles; products
of full 24-bit values next to a value that nearly cancels them, which need every
part and every product of parts; inputs outside the split's range; and the
fragile-flip rule of every fp32 kernel."""
from __future__ import annotations

import numpy as np
import pytest

import hd_inputs
import oracle
from gpu_util import announce, check_against_oracle, dev, torch_or_skip

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hd():
    torch_or_skip()
    import paper_2506_09282_amd as m
    return m


def wide_ints(N, F, D, K, seed):
    """X up to 2^11, B up to 2^6 / F-dependent, C up to 2^9: X and C of two parts,
    sums below 2^24."""
    g = np.random.default_rng(seed)
    bmax = max(1, min(64, (1 << 24) // (F * 2048)))
    X = g.integers(-2047, 2048, (N, F)).astype(np.float32)
    B = g.integers(-bmax, bmax + 1, (F, D)).astype(np.float32)
    C = g.integers(-500, 501, (K, D)).astype(np.float32)
    return X, B, C


def near_products(seed, F, D=128):
    """Rows whose product with column n, x b - c, lies 2^-22 of x b from zero, on
    either side; x and b with all three parts, half of them with a middle and a
    trailing part as large as they can be. Returns X, B, C and H[n, n] for n < D
    (C one-hot: S = H). Each of rounding x b to 24 bits and what the split leaves
    out is at most 2^-24 of x b, so the sign of x b - c is that of the exact value.
    Rows past D are scaled copies."""
    g = np.random.default_rng(seed)

    def mantissas():
        m = 1.0 + g.integers(0, 1 << 23, D) * 2.0 ** -23
        # truncation leaves the largest parts below ...11111111b, rounding to
        # nearest below ...01111111b, in both the lower two parts
        top = (g.integers(0, 128, D) << 16) | 0xFF00 | g.integers(0xF0, 0x100, D)
        mid = (g.integers(0, 128, D) << 16) | 0x7F00 | g.integers(0x70, 0x80, D)
        u = np.where(g.random(D) < 0.5, top, mid)
        return np.where(g.random(D) < 0.5, m, 1.0 + u * 2.0 ** -23)

    x, b = (mantissas() * g.choice([-1, 1], D) * 2.0 ** g.integers(-6, 7, D) for _ in range(2))
    p = x * b  # exact: 48 bits
    c = (p * (1 + g.choice([-1, 1], D) * 2.0 ** -22)).astype(np.float32)
    n, f = np.arange(D), np.array([g.choice(F, 2, replace=False) for _ in range(D)])
    X, B = np.zeros((D, F), np.float32), np.zeros((F, D), np.float32)
    X[n, f[:, 0]], X[n, f[:, 1]] = x, 1.0
    B[f[:, 0], n], B[f[:, 1], n] = b, -c
    H = np.where(p >= c.astype(np.float64), 1, -1)
    X = np.concatenate([X, X * np.float32(2.0), X * np.float32(0.125)])
    return X, B, np.eye(D, dtype=np.float32), H


def run_all(hd, X, B, C, y, K):
    """Scores and labels packed and raw, class sums packed and raw."""
    torch = torch_or_skip()
    Xd, Bd, Cd = (torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (X, B, C))
    yd = torch.from_numpy(y).cuda()
    m = hd.pack_model(Bd, Cd)
    out = [hd.infer_packed(Xd, m, return_scores=True), hd.infer(Xd, Bd, Cd, return_scores=True),
           hd.bundle_classes_packed(Xd, m, yd, K), hd.bundle_classes(Xd, Bd, yd, K)]
    torch.cuda.synchronize()
    return out


def check(hd, X, B, C, seed):
    K = C.shape[0]
    y = np.random.default_rng(seed).integers(-1, K + 1, X.shape[0]).astype(np.int32)
    ref, counts = oracle.infer(X, B, C), oracle.bundle(X, B, y, K)["counts"]
    p, r, cp, cr = run_all(hd, X, B, C, y, K)
    for labels, S in (p, r):
        assert np.array_equal(S.cpu().numpy().astype(np.float64), ref["S"])
        assert np.array_equal(labels.cpu().numpy(), ref["y"])
    for c in (cp, cr):
        assert np.array_equal(c.cpu().numpy(), counts)


# one group of 16 features, a ragged group, one chunk of four groups, one
# more; rows of every offset; samples around the 128-sample tile; dimensions
# around a unit and a pass; one, two and four class blocks
@pytest.mark.parametrize("N,F,D,K", [(257, 1, 64, 3), (257, 15, 65, 32), (300, 16, 256, 33),
                                     (384, 17, 257, 64), (385, 63, 320, 65), (300, 64, 500, 128),
                                     (300, 65, 1000, 10), (513, 130, 96, 5), (300, 1277, 300, 26),
                                     # 64- and 128-sample tiles of one class block
                                     (2000, 40, 1100, 3), (4100, 33, 2100, 32)])
def test_integer_bit_exact(hd, N, F, D, K):
    announce(f"x3 N={N} F={F} D={D} K={K}")
    check(hd, *wide_ints(N, F, D, K, N + F), seed=F)


@pytest.mark.parametrize("F", [2, 5, 16, 40, 130])
def test_every_product_of_parts(hd, F):
    announce(f"x3 near products F={F}")
    for seed in range(4):
        X, B, C, H = near_products(seed, F)
        D = C.shape[0]
        n = np.arange(D)
        y = np.concatenate([n, np.full(X.shape[0] - D, -1)]).astype(np.int32)
        p, r, cp, cr = run_all(hd, X, B, C, y, D)
        for _, S in (p, r):
            S = S.cpu().numpy()
            for i in range(0, X.shape[0], D):
                assert np.array_equal(S[n + i, n], H)
        for c in (cp, cr):
            assert np.array_equal(c.cpu().numpy()[n, n], H)


def test_more_tiles_than_compute_units(hd):
    announce("x3 head and rest")
    check(hd, *wide_ints(256 * 128 + 200, 20, 300, 3, 1), seed=1)


@pytest.mark.parametrize("N,F,D,K", [(2000, 300, 300, 33), (1100, 545, 300, 5), (8300, 530, 1000, 33),
                                     (33000, 520, 256, 32), (3001, 129, 500, 128)])
def test_training_sizes(hd, N, F, D, K):
    """Enough work for this kernel (1.5e8 multiply-adds): two and four sample
    tiles per workgroup, ragged last tiles."""
    torch = torch_or_skip()
    announce(f"x3 training N={N} F={F} D={D} K={K}")
    X, B, _ = wide_ints(N, F, D, K, N)
    y = np.random.default_rng(F).integers(-1, K + 1, N).astype(np.int32)
    H = (X.astype(np.float64) @ B.astype(np.float64) >= 0) * 2 - 1
    want = np.zeros((K, D), np.int64)
    for k in range(K):
        want[k] = H[y == k].sum(axis=0)
    Xd, Bd, yd = (torch.from_numpy(a).cuda() for a in (X, B, y))
    for c in (hd.bundle_classes_packed(Xd, hd.pack_model(Bd, K=K), yd, K),
              hd.bundle_classes(Xd, Bd, yd, K)):
        torch.cuda.synchronize()
        assert np.array_equal(c.cpu().numpy(), want)


@pytest.mark.parametrize("where", ["X", "B", "X, huge", "B, huge"])
def test_nan(hd, where):
    """NaN makes the sums of its row or column NaN (HardSign -1) and needs no other
    instruction, unless there is more: here products that overflow."""
    announce(f"x3 NaN in {where}")
    N, F, D, K = 300, 70, 600, 5
    X, B, C = hd_inputs.make_integer_inputs(N, F, D, K, seed=21)
    if "huge" in where:
        # one product per sum, of 16-bit values, beyond 2^136: infinite on the fp32
        # instruction, inf - inf as a sum of parts
        n = np.arange(N)
        one = np.zeros_like(X)
        one[n, n % F] = np.where(X[n, n % F] < 0, -1, 1)
        X, B = one * np.float32(2.0 ** 70 * 1.0078125), B * np.float32(2.0 ** 66 * 1.0234375)
        B[B == 0] = 1.0
    if where.startswith("X"):
        X[[3, 129, 299], [0, 69, 5]] = np.nan
    else:
        B[[0, 69, 5], [1, 300, 599]] = np.nan
    check(hd, X, B, C, seed=21)


@pytest.mark.parametrize("what", ["inf", "tiny row", "huge b"])
def test_training_range(hd, what):
    """The fall back to the fp32 instruction, with tiles after it."""
    torch = torch_or_skip()
    announce(f"x3 training range: {what}")
    N, F, D, K = 5000, 70, 600, 5
    X, B, _ = hd_inputs.make_integer_inputs(N, F, D, K, seed=11)
    if what == "inf":
        B[7] = np.where(B[7] == 0, 1, B[7])
        X[5, 7], X[2000, 7], X[2001, 3] = np.inf, -np.inf, np.nan
    elif what == "tiny row":
        X[1000] *= np.float32(2.0 ** -118)
    else:
        B = B * np.float32(2.0 ** 90)
    y = np.random.default_rng(1).integers(0, K, N).astype(np.int32)
    ref = oracle.bundle(X, B, y, K)["counts"]
    Xd, Bd, yd = (torch.from_numpy(a).cuda() for a in (X, B, y))
    for c in (hd.bundle_classes_packed(Xd, hd.pack_model(Bd, K=K), yd, K),
              hd.bundle_classes(Xd, Bd, yd, K)):
        torch.cuda.synchronize()
        assert np.array_equal(c.cpu().numpy(), ref)


def test_row_offsets_of_x(hd):
    """X 4-byte aligned only."""
    torch = torch_or_skip()
    X, B, C = wide_ints(300, 50, 300, 4, 2)
    buf = torch.zeros(X.size + 1, device="cuda")
    buf[1:] = torch.from_numpy(X.reshape(-1)).cuda()
    y, S = hd.infer(buf[1:].view(300, 50), torch.from_numpy(B).cuda(), torch.from_numpy(C).cuda(),
                    return_scores=True)
    torch.cuda.synchronize()
    ref = oracle.infer(X, B, C)
    assert np.array_equal(S.cpu().numpy().astype(np.float64), ref["S"])
    assert np.array_equal(y.cpu().numpy(), ref["y"])


# Inputs that the split cannot take: the pass falls back to the fp32
# instruction. Powers of two keep every sum exact.
@pytest.mark.parametrize("what", ["inf", "huge x", "tiny x", "tiny row", "huge b", "tiny column",
                                  "huge c", "tiny c", "zero row and column"])
def test_range(hd, what):
    announce(f"x3 range: {what}")
    N, F, D, K = 300, 70, 600, 5
    X, B, C = hd_inputs.make_integer_inputs(N, F, D, K, seed=9)
    if what == "inf":
        B[7] = np.where(B[7] == 0, 1, B[7])
        X[5, 7], X[200, 7], X[201, 3] = np.inf, -np.inf, np.nan
    elif what == "huge x":
        X = X * np.float32(2.0 ** 90)
    elif what == "tiny x":
        X = X * np.float32(2.0 ** -118)
    elif what == "tiny row":
        X[100] *= np.float32(2.0 ** -118)
    elif what == "huge b":
        B = B * np.float32(2.0 ** 90)
    elif what == "tiny column":
        B[:, 300] *= np.float32(2.0 ** -118)
    elif what == "huge c":
        C = C * np.float32(2.0 ** 90)
    elif what == "tiny c":
        C = C * np.float32(2.0 ** -118)
    else:
        X[50] = 0
        B[:, 40] = 0
    check(hd, X, B, C, seed=9)


@pytest.mark.parametrize("side", ["X", "B"])
def test_parts_that_do_not_exist(hd, side):
    """Values with bits below 2^-133, which have no three parts, beside ordinary
    ones that meet zeros: every row and column has its largest magnitude at 1 or
    more, and the sums are those of the small values alone (exact: integers below
    2^24 times 2^-149 and 2^-134)."""
    announce(f"x3 missing parts of {side}")
    N, F, D, K = 300, 40, 600, 5
    g = np.random.default_rng(13)
    for scale in (2.0 ** -149, 2.0 ** -134):
        small = g.integers(-1000, 1001, (N, F) if side == "X" else (F, D)) * scale
        other = g.integers(-1, 2, (F, D) if side == "X" else (N, F)).astype(np.float64)
        X, B = (small, other) if side == "X" else (other, small)
        X[:, 0], B[0], X[:, 1], B[1] = 3.0, 0.0, 0.0, 5.0
        C = g.integers(-500, 501, (K, D)).astype(np.float32)
        check(hd, X.astype(np.float32), B.astype(np.float32), C, seed=13)


def test_neighbours_do_not_matter(hd):
    """Sums within rounding of zero, whose signs the two instructions take
    differently: a row or a column that needs the fp32 instruction changes no
    other row's or column's signs."""
    announce("x3 neighbours")
    N, F, D, K = 384, 48, 8256, 5
    g = np.random.default_rng(17)
    x = g.standard_normal(F).astype(np.float32)
    x[-1] = 1.0
    X = (x * 2.0 ** g.integers(-3, 4, (N, 1))).astype(np.float32)
    B = g.standard_normal((F, D)).astype(np.float32)
    B[-1] = -(x[:-1].astype(np.float64) @ B[:-1].astype(np.float64))
    C = g.integers(-500, 501, (K, D)).astype(np.float32)
    y = g.integers(0, K, N).astype(np.int32)
    y[7] = -1
    base = [t if isinstance(t, tuple) else (t,) for t in run_all(hd, X, B, C, y, K)]
    rows, cols = np.arange(N) != 7, np.arange(D) != 300
    for what in ("row", "column"):
        X2, B2, C2 = X.copy(), B.copy(), C.copy()
        if what == "row":
            X2[7, 3] = np.inf
        else:
            B2[5, 300] = np.inf
            C2[:, 300] = 0
            base = [t if isinstance(t, tuple) else (t,) for t in run_all(hd, X, B, C2, y, K)]
        got = [t if isinstance(t, tuple) else (t,) for t in run_all(hd, X2, B2, C2, y, K)]
        for k in range(2):  # packed, raw
            for a, b in zip(base[k], got[k]):
                a, b = a.cpu().numpy(), b.cpu().numpy()
                assert np.array_equal(a[rows] if what == "row" else a,
                                      b[rows] if what == "row" else b), (what, k)
            a, b = base[2 + k][0].cpu().numpy(), got[2 + k][0].cpu().numpy()
            assert np.array_equal(a if what == "row" else a[:, cols],
                                  b if what == "row" else b[:, cols]), (what, k)


@pytest.mark.parametrize("N,F,D", [(1500, 561, 2048), (700, 21, 256), (3000, 600, 2816)])
def test_training_in_chunks(hd, N, F, D):
    """The counts of one call bit for bit, from chunks of all sizes, on sums
    within rounding of zero (every row a multiple of one, the last row of B
    cancels it): which sign such a sum takes depends on the kernel, so it must
    not depend on the chunk."""
    torch = torch_or_skip()
    announce(f"x3 training in chunks N={N} F={F} D={D}")
    K, g = 4, np.random.default_rng(N)
    x = g.standard_normal(F).astype(np.float32)
    x[-1] = 1.0
    X = (x * 2.0 ** g.integers(-3, 4, (N, 1))).astype(np.float32)
    B = g.standard_normal((F, D)).astype(np.float32)
    B[-1] = -(x[:-1].astype(np.float64) @ B[:-1].astype(np.float64))
    Xd, Bd = torch.from_numpy(X).cuda(), torch.from_numpy(B).cuda()
    yd = torch.from_numpy(g.integers(0, K, N).astype(np.int32)).cuda()
    m = hd.pack_model(Bd, K=K)
    for call in (lambda *a, **k: hd.bundle_classes_packed(a[0], m, *a[1:], **k),
                 lambda *a, **k: hd.bundle_classes(a[0], Bd, *a[1:], **k)):
        one = call(Xd, yd, K)
        for cuts in ((1, 60, 245), (33, 34, 161, 400), (N - 1,)):
            counts = torch.zeros_like(one)
            for a, b in zip((0,) + cuts, cuts + (N,)):
                call(Xd[a:b], yd[a:b], K, counts=counts)
            torch.cuda.synchronize()
            assert torch.equal(one, counts), cuts


@pytest.mark.parametrize("N,F,D,K,dist", [(512, 784, 2048, 10, "uniform01_zero20"),
                                          (512, 617, 1500, 26, "normal"),
                                          (300, 3000, 700, 40, "uniform_pm1")])
def test_error_within_fp32_bound(hd, N, F, D, K, dist):
    """The fragile-flip rule of every fp32 kernel (an error bound of F roundings
    to 24 bits), which a product with fewer than all its parts would break."""
    announce(f"x3 real N={N} F={F} D={D} K={K}")
    X, B, C = hd_inputs.make_inputs(N, F, D, K, dist, seed=4)
    torch = torch_or_skip()
    for out in (hd.infer_packed(dev(X, "f32"), hd.pack_model(dev(B, "f32"), dev(C, "f32")),
                                return_scores=True),
                hd.infer(dev(X, "f32"), dev(B, "f32"), dev(C, "f32"), return_scores=True)):
        torch.cuda.synchronize()
        rep, _ = check_against_oracle(X, B, C, out[0].cpu().numpy(),
                                      out[1].cpu().numpy().astype(np.float64))
        assert rep["ok"], rep
