"""64 < N <= 128 samples on a packed bf16 or int8 model in one call of the
fragment kernel (two passes of 64): bit-exact on integer inputs at the edges of
its passes, in both reduction modes, and within the workspace of 64-sample calls."""
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


# a second pass of one row, of 16 and 17, whole; the shortest rows; rows of
# every rows-per-lane size, with X in registers and read in every step; three
# blocks per workgroup and workgroups without a block; the most classes; 250 =
# 128 + 122; rows too long for two passes (64-sample calls)
CASES = [(65, 16, 64, 2), (80, 17, 300, 6), (81, 191, 1000, 16), (127, 300, 1500, 5),
         (128, 561, 10240, 6), (100, 576, 12288, 3), (128, 700, 2000, 16), (250, 561, 2048, 6),
         (128, 1000, 1500, 5), (100, 15, 100, 3)]


@pytest.mark.parametrize("det", [False, True])
@pytest.mark.parametrize("dtype", ["bf16", "i8"])
@pytest.mark.parametrize("N,F,D,K", CASES)
def test_integer_bit_exact(hd, N, F, D, K, dtype, det):
    torch = torch_or_skip()
    announce(f"two pass {dtype} N={N} F={F} D={D} K={K} det={det}")
    X, B, C = hd_inputs.make_integer_inputs(N, F, D, K, seed=N + F)
    tdt = torch.bfloat16 if dtype == "bf16" else torch.int8
    Xd, Bd, Cd = (torch.from_numpy(a).cuda().to(tdt) for a in (X, B, C))
    m, ref = hd.pack_model(Bd, Cd), oracle.infer(X, B, C)
    full = int(hd.lib().hd_infer_packed_workspace_bytes(N, F, D, K, m.dt))
    # what 64-sample calls need: counters, then 32 replicas or one per block and group
    least = 256 * 9 + 4 * 64 * K * (-(-D // 16) + 8 if det else 32)
    sizes = [full] if dtype == "i8" else sorted({least, full})
    for nbytes in sizes:
        ws = torch.zeros(nbytes, dtype=torch.uint8, device="cuda")
        y = torch.empty(N, dtype=torch.int32, device="cuda")
        S = torch.empty((N, K), dtype=torch.float32, device="cuda")
        for _ in range(2):
            hd.infer_packed(Xd, m, out=(y, S), workspace=ws, deterministic=det)
            torch.cuda.synchronize()
            assert np.array_equal(S.cpu().numpy().astype(np.float64), ref["S"])
            assert np.array_equal(y.cpu().numpy(), ref["y"])
            assert int(ws.count_nonzero()) == 0
    y, S = hd.infer_packed_noalloc(Xd, m, return_scores=True)
    torch.cuda.synchronize()
    assert np.array_equal(S.cpu().numpy().astype(np.float64), ref["S"])
    assert np.array_equal(y.cpu().numpy(), ref["y"])


# X as a slice of a larger tensor: 2-byte aligned only (64-sample calls of the
# kernel that reads it so); the whole calls, the noalloc one included
@pytest.mark.parametrize("det", [False, True])
@pytest.mark.parametrize("shift", [1, 2, 4])
@pytest.mark.parametrize("N", [65, 100, 128, 250])
def test_unaligned_bf16_x(hd, N, shift, det):
    torch = torch_or_skip()
    F, D, K = 561, 1000, 6
    announce(f"two pass, X shifted by {shift} N={N} det={det}")
    X, B, C = hd_inputs.make_integer_inputs(N, F, D, K, seed=N)
    buf = torch.zeros(N * F + shift, dtype=torch.bfloat16, device="cuda")
    buf[shift:] = torch.from_numpy(X.reshape(-1)).cuda().to(torch.bfloat16)
    Xd = buf[shift:].view(N, F)
    m = hd.pack_model(*(torch.from_numpy(a).cuda().to(torch.bfloat16) for a in (B, C)))
    ref = oracle.infer(X, B, C)
    for call in (hd.infer_packed, hd.infer_packed_noalloc):
        y, S = call(Xd, m, return_scores=True, deterministic=det)
        torch.cuda.synchronize()
        assert np.array_equal(S.cpu().numpy().astype(np.float64), ref["S"])
        assert np.array_equal(y.cpu().numpy(), ref["y"])
