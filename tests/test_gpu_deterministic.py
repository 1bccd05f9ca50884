"""GPU: the deterministic mode (HD_DETERMINISTIC). Repeated calls give
bit-identical scores and labels on every small-batch kernel (whose default
mode sums partial scores with fp32 atomics in arrival order) and on the
large-batch path; the results stay within the oracle rule, are bit-exact on
integer inputs, and leave the workspace reusable by either mode."""
import numpy as np
import pytest

import hd_inputs
import oracle
from gpu_util import RTOL, announce, check_against_oracle, dev, torch_or_skip

pytestmark = pytest.mark.gpu

REPEATS = 20


@pytest.fixture(scope="module")
def hd():
    torch_or_skip()
    import paper_2506_09282_amd as hd
    hd.lib()
    return hd


# (N, F, D, K, dtype, packed, kernel): every small-batch kernel, the chunked
# small route and both large-batch kernels.
CASES = [
    (1, 561, 10240, 6, "f32", False, "small_flat_kernel"),
    (4, 561, 2048, 6, "bf16", True, "small_flat_kernel"),
    (16, 33, 1000, 5, "f32", False, "small_block_mfma_kernel"),
    (16, 3072, 1000, 5, "f32", False, "small_valu_kernel"),
    (64, 33, 1000, 5, "f32", False, "small_mfma_kernel"),
    (32, 561, 10240, 6, "f32", True, "small_frag_mfma_kernel"),
    (64, 617, 10240, 26, "f32", True, "small_valu_kernel"),
    (200, 561, 10240, 6, "f32", True, "small_frag_mfma_kernel"),  # 64-sample calls, two passes
    (32, 561, 10240, 6, "bf16", True, "small_frag_mfma_kernel"),
    (16, 617, 4096, 26, "bf16", True, "large_fused_kernel"),
    (16, 3072, 1000, 5, "bf16", False, "large_chunked_dma_kernel"),
    (32, 561, 20480, 6, "f32", True, "small_frag_mfma_kernel"),  # the fragment kernel's B ring
]
# the small-batch cases (integer inputs are exact for them in any order)
SMALL_CASES = CASES[:9] + CASES[11:]


def run(hd, Xd, Bd, Cd, packed, det, model=None):
    if packed:
        return hd.infer_packed(Xd, model, return_scores=True, deterministic=det)
    return hd.infer(Xd, Bd, Cd, return_scores=True, deterministic=det)


@pytest.mark.parametrize("N,F,D,K,dtype,packed,kernel", CASES)
def test_deterministic_repeats_bit_identical(hd, N, F, D, K, dtype, packed, kernel):
    torch = torch_or_skip()
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    assert hd.infer_kernel(min(N, 64), F, D, K, tdt, packed=packed) == kernel
    announce(f"deterministic {kernel} {dtype} N={N} F={F} D={D} K={K} packed={packed}")
    X, B, C = hd_inputs.make_inputs(N, F, D, K, "uniform_pm1", seed=N + K, dtype=dtype)
    Xd, Bd, Cd = dev(X, dtype), dev(B, dtype), dev(C, dtype)
    model = hd.pack_model(Bd, Cd) if packed else None
    y0, S0 = run(hd, Xd, Bd, Cd, packed, True, model)
    for i in range(REPEATS):
        # interleave default-mode calls on the same cached workspace
        run(hd, Xd, Bd, Cd, packed, False, model)
        y, S = run(hd, Xd, Bd, Cd, packed, True, model)
        torch.cuda.synchronize()
        assert torch.equal(y, y0), i
        assert torch.equal(S, S0), i
    rep, _ = check_against_oracle(X, B, C, y0.cpu().numpy(), S0.cpu().numpy().astype(np.float64),
                                  rtol=RTOL)
    assert rep["ok"], rep


@pytest.mark.parametrize("N,F,D,K,dtype,packed,kernel", SMALL_CASES)
def test_deterministic_integer_bit_exact(hd, N, F, D, K, dtype, packed, kernel):
    """Small integers: every sum is exact in any order, so the fixed-order
    reduction must reproduce the oracle bit for bit."""
    torch = torch_or_skip()
    announce(f"deterministic integer {kernel} N={N}")
    X, B, C = hd_inputs.make_integer_inputs(N, F, D, K, seed=N + F)
    Xd, Bd, Cd = dev(X, dtype), dev(B, dtype), dev(C, dtype)
    model = hd.pack_model(Bd, Cd) if packed else None
    y, S = run(hd, Xd, Bd, Cd, packed, True, model)
    torch.cuda.synchronize()
    ref = oracle.infer(X, B, C)
    assert np.array_equal(S.cpu().numpy().astype(np.float64), ref["S"])
    assert np.array_equal(y.cpu().numpy(), ref["y"])


def test_deterministic_noalloc(hd):
    torch = torch_or_skip()
    N, F, D, K = 32, 561, 10240, 6
    X, B, C = hd_inputs.make_inputs(N, F, D, K, "uniform_pm1", seed=2)
    Xd = dev(X, "f32")
    model = hd.pack_model(dev(B, "f32"), dev(C, "f32"))
    y0, S0 = hd.infer_packed_noalloc(Xd, model, return_scores=True, deterministic=True)
    y1, S1 = hd.infer_packed(Xd, model, return_scores=True, deterministic=True)
    for _ in range(5):
        y2, S2 = hd.infer_packed_noalloc(Xd, model, return_scores=True, deterministic=True)
        torch.cuda.synchronize()
        assert torch.equal(S2, S0) and torch.equal(y2, y0)
    assert torch.equal(S1, S0) and torch.equal(y1, y0)


# The split of D of the large-batch kernels follows the workspace, in the default
# mode; two 64-sample calls or one of 128 likewise.
@pytest.mark.parametrize("N,F,D,K,dtype", [(4096, 617, 10240, 26, "bf16"),
                                           (300, 784, 10240, 10, "bf16"),
                                           (2500, 300, 10240, 20, "f32"),
                                           (900, 1500, 4096, 40, "f32"),
                                           (100, 561, 10240, 6, "bf16"),
                                           (250, 300, 5000, 10, "bf16")])
def test_deterministic_whatever_the_workspace(hd, N, F, D, K, dtype):
    """The same bits from the least workspace that a call takes, the size
    query's, a larger one and the library's own scratch."""
    torch = torch_or_skip()
    announce(f"deterministic workspaces {dtype} N={N} F={F} D={D} K={K}")
    X, B, C = hd_inputs.make_inputs(N, F, D, K, "uniform_pm1", seed=N, dtype=dtype)
    Xd, Bd, Cd = dev(X, dtype), dev(B, dtype), dev(C, dtype)
    m = hd.pack_model(Bd, Cd)
    out = (torch.empty(N, dtype=torch.int32, device="cuda"),
           torch.empty((N, K), dtype=torch.float32, device="cuda"))

    def call(ws, raw):
        a = (Xd, Bd, Cd) if raw else (Xd, m)
        (hd.infer if raw else hd.infer_packed)(*a, out=out, workspace=ws, deterministic=True)
        torch.cuda.synchronize()
        return out[0].clone(), out[1].clone()

    for raw in (False, True):
        L = hd.lib()
        query = L.hd_infer_workspace_bytes if raw else L.hd_infer_packed_workspace_bytes
        full = int(query(N, F, D, K, m.dt))
        ws = torch.zeros(2 * full + 256, dtype=torch.uint8, device="cuda")
        want = call(ws[:full], raw)
        lo, hi = 0, full  # the least size: below it the call is refused
        while hi - lo > 256:
            mid = (lo + hi) // 2 // 256 * 256
            try:
                call(ws[:mid], raw)
                hi = mid
            except hd.HDError as e:
                assert e.status == hd.HD_ERR_WORKSPACE
                lo = mid
        for nbytes in (hi, (hi + full) // 2, 2 * full):
            got = call(ws[:nbytes], raw)
            assert torch.equal(got[1], want[1]) and torch.equal(got[0], want[0]), (raw, nbytes)
        if not raw:
            try:
                got = hd.infer_packed_noalloc(Xd, m, return_scores=True, deterministic=True)
            except hd.HDError as e:  # more than the scratch at least
                assert e.status == hd.HD_ERR_WORKSPACE
                continue
            torch.cuda.synchronize()
            assert torch.equal(got[1], want[1]) and torch.equal(got[0], want[0])
