"""The large-batch kernel that holds X in registers (bf16, int8) and the
second launch that sums the slices of a split D: bit-exact on integer inputs
at the edges of its tiles, and on the calls whose workspace is smaller than the
size query's answer."""
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
    """Device copy whose first element lies `shift` elements past a 256-byte boundary."""
    torch = torch_or_skip()
    t = torch.from_numpy(np.ascontiguousarray(a)).cuda().to(
        torch.bfloat16 if dtype == "bf16" else torch.int8)
    buf = torch.zeros(t.numel() + shift, dtype=t.dtype, device="cuda")
    buf[shift:] = t.reshape(-1)
    return buf[shift:].view(t.shape)


def model(F, D, K, seed):
    _, B, C = hd_inputs.make_integer_inputs(1, F, D, K, seed=seed)
    return B, C


def check(X, B, C, y, S, rows=None):
    ref = oracle.infer(X, B, C, rows=rows)
    y, S = y.cpu().numpy(), S.cpu().numpy()
    if rows is not None:
        y, S = y[rows], S[rows]
    assert np.array_equal(S.astype(np.float64), ref["S"])
    assert np.array_equal(y, ref["y"])


# one f-step, a full and a ragged last f-step, the most steps for each count
# of class blocks; odd rows; the first and last class of a block; rows 1, 255,
# 256, 257 of the 256-sample tile; D not a multiple of 32; D of one unit
CASES = [("bf16", 65, 1, 100, 33), ("bf16", 257, 127, 1000, 32), ("bf16", 256, 128, 96, 1),
         ("bf16", 255, 639, 1500, 26), ("bf16", 513, 640, 64, 10), ("bf16", 300, 511, 777, 33),
         ("bf16", 300, 512, 777, 64), ("bf16", 300, 319, 500, 65), ("bf16", 300, 320, 500, 128),
         ("i8", 257, 31, 1000, 32), ("i8", 255, 1279, 500, 5), ("i8", 513, 1280, 64, 10),
         ("i8", 300, 1023, 333, 64), ("i8", 300, 639, 333, 100), ("i8", 300, 33, 100, 17),
         ("i8", 300, 618, 512, 3),
         # rows of 41 to 49 f-steps: a part of X in LDS, slots of half a unit
         ("bf16", 257, 641, 96, 32), ("bf16", 300, 784, 1000, 10), ("bf16", 513, 783, 500, 5),
         ("bf16", 255, 705, 333, 7), ("i8", 300, 1281, 96, 32), ("i8", 300, 1568, 333, 10),
         ("i8", 257, 1567, 64, 7),
         # D in up to 64 slices, summed by one to four groups; the fewest samples
         ("bf16", 65, 128, 4096, 33), ("i8", 70, 64, 2500, 17), ("bf16", 17, 690, 4096, 20),
         ("bf16", 16, 690, 4096, 20)]


@pytest.mark.parametrize("dtype,N,F,D,K", CASES)
def test_integer_bit_exact(hd, dtype, N, F, D, K):
    torch = torch_or_skip()
    announce(f"xreg {dtype} N={N} F={F} D={D} K={K}")
    X, B, C = hd_inputs.make_integer_inputs(N, F, D, K, seed=N + F)
    m = hd.pack_model(up(B, dtype), up(C, dtype))
    Xd = up(X, dtype)
    for _ in range(2):  # the workspace is left zeroed
        y, S = hd.infer_packed(Xd, m, return_scores=True)
        torch.cuda.synchronize()
        check(X, B, C, y, S)
    y, S = hd.infer(Xd, up(B, dtype), up(C, dtype), return_scores=True)
    torch.cuda.synchronize()
    check(X, B, C, y, S)


def test_more_tiles_than_compute_units(hd):
    """Whole rounds of tiles run unsplit, the tiles left over in a second launch."""
    torch = torch_or_skip()
    N, F, D, K = 65536 + 300, 17, 320, 5
    announce(f"xreg head and rest N={N}")
    X, B, C = hd_inputs.make_integer_inputs(N, F, D, K, seed=3)
    y, S = hd.infer_packed(up(X, "bf16"), hd.pack_model(up(B, "bf16"), up(C, "bf16")),
                           return_scores=True)
    torch.cuda.synchronize()
    check(X, B, C, y, S)


@pytest.mark.parametrize("dtype,shift", [("bf16", 2), ("bf16", 1), ("i8", 4), ("i8", 1)])
def test_x_alignment(hd, dtype, shift):
    """X 4-byte aligned (this kernel) and not (the kernels with X in LDS)."""
    torch = torch_or_skip()
    N, F, D, K = 300, 101, 500, 9
    announce(f"xreg X shifted by {shift} {dtype}")
    X, B, C = hd_inputs.make_integer_inputs(N, F, D, K, seed=4)
    y, S = hd.infer_packed(up(X, dtype, shift), hd.pack_model(up(B, dtype), up(C, dtype)),
                           return_scores=True)
    torch.cuda.synchronize()
    check(X, B, C, y, S)


@pytest.mark.parametrize("dtype", ["bf16", "i8"])
def test_small_workspace(hd, dtype):
    """The split of D follows the workspace: what suffices for the kernels with
    X in LDS (128-sample tiles, slices that fill 256 compute units) suffices."""
    torch = torch_or_skip()
    N, F, D, K = 2000, 300, 4096, 10
    X, B, C = hd_inputs.make_integer_inputs(N, F, D, K, seed=5)
    m, Xd = hd.pack_model(up(B, dtype), up(C, dtype)), up(X, dtype)
    least = 256 + 16 * N * K * 4  # 16 tiles of 128 samples, 16 slices
    full = hd.lib().hd_infer_packed_workspace_bytes(N, F, D, K, m.dt)
    for nbytes in (least, max(least, full)):
        announce(f"xreg {dtype} workspace {nbytes}")
        guard = 4096
        buf = torch.zeros(nbytes + guard, dtype=torch.uint8, device="cuda")
        buf[nbytes:] = 0xA5
        y = torch.empty(N, dtype=torch.int32, device="cuda")
        S = torch.empty((N, K), dtype=torch.float32, device="cuda")
        hd.infer_packed(Xd, m, out=(y, S), workspace=buf[:nbytes])
        torch.cuda.synchronize()
        check(X, B, C, y, S)
        assert bool((buf[nbytes:] == 0xA5).all()) and int(buf[:nbytes].count_nonzero()) == 0
    y, S = hd.infer_packed_noalloc(Xd, m, return_scores=True)
    torch.cuda.synchronize()
    check(X, B, C, y, S)


def test_infinite_and_nan_features(hd):
    """A row's infinities and NaNs stay in the row, whatever its neighbours'
    rows and the padding past F hold."""
    torch = torch_or_skip()
    N, F, D, K = 300, 37, 256, 4
    announce("xreg inf and nan")
    X, B, C = hd_inputs.make_integer_inputs(N, F, D, K, seed=6)
    B[5] = np.where(B[5] == 0, 1, B[5])
    X[3, 5], X[70, 5], X[120, 36], X[121, 0] = np.inf, -np.inf, np.nan, np.nan
    y, S = hd.infer_packed(up(X, "bf16"), hd.pack_model(up(B, "bf16"), up(C, "bf16")),
                           return_scores=True)
    torch.cuda.synchronize()
    check(X, B, C, y, S)
