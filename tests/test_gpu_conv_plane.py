"""Convolutions of many positions whose input rows stay in LDS (gemm_conv_plane.hip): six taps or more, dense planes, channels in
whole blocks of 32.  Small integers: every sum is exact, so the result must be the oracle's bit for bit."""
import numpy as np
import pytest
import torch

import paper_2507_11978_amd as nt
import synthetic_inputs as si
from oracle import numeric as onum
from gpu_util import TORCH_DT, inside, to_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,stride,pad", [
    # one shape for each kernel that is built, all its tiles of one height: 9 taps, 256 filters per program ...
    ((19, 64, 57, 57, 130, 3, 3), (1, 1), (1, 1)),     # tiles of 256 positions; planes of odd size: 2-byte aligned runs
    ((18, 64, 48, 48, 130, 3, 3), (1, 1), (1, 1)),     # 192
    ((21, 64, 40, 40, 130, 3, 3), (1, 1), (1, 1)),     # 160
    ((18, 64, 40, 40, 130, 3, 3), (1, 1), (1, 1)),     # 128
    ((9, 64, 48, 48, 130, 3, 3), (1, 1), (1, 1)),      # 96
    ((30, 32, 56, 56, 160, 3, 3), (2, 2), (1, 1)),     # 96, one set of planes; one block of channels
    # ... 128 filters
    ((8, 64, 56, 56, 130, 3, 3), (1, 1), (1, 1)),
    ((18, 64, 48, 48, 72, 3, 3), (1, 1), (1, 1)),
    ((21, 32, 28, 28, 130, 3, 3), (1, 1), (1, 1)),
    ((31, 32, 20, 20, 130, 3, 3), (1, 1), (1, 1)),
    ((26, 32, 20, 20, 72, 3, 3), (1, 1), (1, 1)),
    ((32, 32, 56, 56, 72, 3, 3), (2, 2), (1, 1)),
    # other numbers of taps
    ((21, 32, 40, 40, 130, 5, 5), (1, 1), (2, 2)),
    ((15, 32, 33, 33, 130, 5, 5), (1, 1), (2, 2)),
    ((19, 32, 57, 57, 130, 5, 5), (1, 1), (2, 2)),
    ((11, 32, 56, 56, 130, 5, 5), (1, 1), (2, 2)),
    ((6, 64, 56, 56, 130, 5, 5), (1, 1), (2, 2)),
    ((30, 32, 33, 33, 72, 5, 5), (1, 1), (2, 2)),
    ((34, 32, 17, 17, 72, 5, 5), (1, 1), (2, 2)),
    ((11, 32, 56, 56, 72, 5, 5), (1, 1), (2, 2)),
    # odd numbers of blocks of channels, taps in two rows of three, strides and padding of their own, rows of odd length
    ((9, 96, 48, 48, 130, 3, 3), (1, 1), (0, 2)),
    ((16, 96, 41, 37, 130, 2, 3), (1, 1), (1, 0)),
    ((20, 96, 47, 47, 200, 3, 3), (2, 1), (1, 1)),
    ((150, 64, 9, 9, 136, 3, 3), (1, 1), (1, 1)),      # several images in a tile
])
def test_conv_plane(shape, stride, pad):
    N, C, H, W, F, R, S = shape
    for dt, out, lead in (("f16", "f16", 33), ("bf16", "f32", 32)):
        X, Wt = si.conv_inputs(N, C, H, W, F, R, S, dt, seed=93, dist="int")
        ref = onum.conv2d(X, Wt, dt, stride, pad, nthreads=16)
        want = torch.from_numpy(ref).to(torch.float32).to(TORCH_DT[out])
        x, w = inside(to_gpu(X, dt), lead), inside(to_gpu(Wt, dt), 32)
        big = torch.full((N, F + 3, ref.shape[2], ref.shape[3]), float("nan"), dtype=TORCH_DT[out], device="cuda")
        Y = big[:, 2:F + 2]
        nt.conv2d_implicit(x, w, Y, stride, pad)
        torch.cuda.synchronize()
        assert nt.last_conv_plan().kernel == nt.CONV_MANY_POSITIONS
        assert nt.last_kernel_path() == (nt.PATH_CONV_TAP if stride == (1, 1) else nt.PATH_CONV_CL) and nt.last_k_split() == 1
        assert torch.equal(Y.cpu(), want), (shape, stride, pad, dt, out)
        assert torch.isnan(big[:, :2]).all() and torch.isnan(big[:, F + 2:]).all()


@pytest.mark.parametrize("positions,filters,runs,tiles,shape,stride,pad", [
    # ... and one whose tiles have both heights (9 taps, then any number)
    ((256, 224), 256, 2, (256, 249), (36, 32, 58, 58, 130, 3, 3), (1, 1), (1, 1)),
    ((224, 192), 256, 2, (85, 83), (64, 32, 60, 9, 520, 3, 3), (1, 1), (1, 1)),
    ((192, 160), 256, 2, (256, 218), (38, 64, 48, 48, 130, 3, 3), (1, 1), (1, 0)),
    ((160, 128), 256, 2, (256, 198), (38, 64, 30, 58, 130, 3, 3), (1, 1), (1, 1)),
    ((128, 96), 256, 2, (256, 256), (28, 96, 64, 64, 200, 3, 3), (2, 1), (1, 1)),
    ((128, 96), 256, 3, (256, 203), (51, 64, 64, 64, 160, 3, 3), (2, 2), (1, 1)),
    ((256, 224), 128, 2, (256, 255), (58, 64, 50, 44, 40, 3, 3), (1, 1), (0, 1)),
    ((224, 192), 128, 2, (85, 73), (49, 64, 56, 14, 300, 3, 3), (1, 1), (1, 0)),
    ((192, 160), 128, 2, (512, 231), (33, 96, 64, 64, 72, 3, 3), (1, 1), (1, 1)),
    ((160, 128), 128, 2, (256, 242), (58, 96, 62, 40, 100, 3, 3), (1, 2), (1, 1)),
    ((128, 96), 128, 2, (256, 229), (53, 96, 38, 56, 128, 3, 3), (1, 2), (1, 0)),
    ((128, 96), 128, 3, (256, 227), (55, 96, 64, 64, 40, 3, 3), (2, 2), (0, 1)),
    ((192, 160), 256, 2, (256, 210), (47, 32, 44, 44, 130, 5, 5), (1, 1), (2, 0)),
    ((256, 224), 256, 3, (128, 124), (49, 32, 44, 28, 390, 7, 1), (1, 1), (3, 0)),
    ((192, 160), 256, 3, (256, 248), (44, 96, 64, 64, 136, 3, 2), (2, 1), (1, 0)),
    ((128, 96), 256, 3, (256, 220), (51, 96, 64, 64, 100, 3, 2), (2, 2), (1, 1)),
    ((256, 224), 128, 2, (256, 233), (50, 32, 48, 49, 40, 3, 5), (1, 1), (1, 2)),
    ((256, 224), 128, 3, (256, 245), (49, 32, 50, 53, 40, 5, 5), (1, 1), (2, 0)),
    # (the two kernels for which the estimate never mixes its heights: one each)
    ((128, 96), 256, 2, (241, 0), (63, 32, 22, 22, 130, 3, 5), (1, 1), (1, 2)),
    ((128, 96), 256, 2, (0, 180), (43, 64, 20, 20, 130, 7, 1), (1, 1), (3, 0)),
    ((128, 96), 128, 2, (204, 0), (57, 64, 32, 14, 40, 3, 2), (1, 1), (0, 1)),
    ((128, 96), 128, 2, (0, 104), (29, 32, 18, 18, 40, 4, 3), (1, 1), (2, 1)),
])
def test_conv_plane_tiles_of_two_heights(positions, filters, runs, tiles, shape, stride, pad):
    """Both heights that a kernel is built for, and where the second takes over.  The reference is the oracle's product over the unfolded
    input; the last image's, where the ragged last tile lies, is checked against its direct convolution."""
    N, C, H, W, F, R, S = shape
    dt, out = ("f16", "f16") if positions[0] % 64 else ("bf16", "f32")
    X, Wt = si.conv_inputs(N, C, H, W, F, R, S, dt, seed=95, dist="int")
    P, Q = (H + 2 * pad[0] - R) // stride[0] + 1, (W + 2 * pad[1] - S) // stride[1] + 1
    Xp = np.zeros((N, C, H + 2 * pad[0], W + 2 * pad[1]), dtype=np.uint16)
    Xp[:, :, pad[0]:pad[0] + H, pad[1]:pad[1] + W] = X
    U = np.stack([Xp[:, :, r:r + (P - 1) * stride[0] + 1:stride[0], s:s + (Q - 1) * stride[1] + 1:stride[1]] for r in range(R) for s in range(S)], axis=2)
    ref = onum.gemm(np.ascontiguousarray(U.transpose(0, 3, 4, 1, 2).reshape(N * P * Q, C * R * S)), np.ascontiguousarray(Wt.reshape(F, C * R * S).T), dt, nthreads=16)
    ref = ref.reshape(N, P * Q, F).transpose(0, 2, 1).reshape(N, F, P, Q)
    assert np.array_equal(onum.conv2d(X[N - 1:], Wt[:8], dt, stride, pad, nthreads=16)[0], ref[N - 1, :8])
    big = torch.full((N, F + 3, P, Q), float("nan"), dtype=TORCH_DT[out], device="cuda")
    Y = big[:, 2:F + 2]
    nt.conv2d_implicit(inside(to_gpu(X, dt), 33), to_gpu(Wt, dt), Y, stride, pad)
    torch.cuda.synchronize()
    plan = nt.last_conv_plan()
    assert plan.kernel == nt.CONV_MANY_POSITIONS
    assert (tuple(plan.positions), plan.filters, plan.runs, tuple(plan.tiles)) == (positions, filters, runs, tiles)
    assert torch.equal(Y.cpu(), torch.from_numpy(ref).to(torch.float32).to(TORCH_DT[out]))
    assert torch.isnan(big[:, :2]).all() and torch.isnan(big[:, F + 2:]).all()


@pytest.mark.parametrize("shape,stride", [((9, 64, 48, 48, 130, 3, 3), 1), ((30, 32, 56, 56, 160, 3, 3), 2), ((4, 96, 14, 14, 64, 3, 3), 1)])
def test_conv_resident_keeps_an_infinity_to_its_window(shape, stride):
    """An infinity and a NaN in the input reach the outputs whose windows hold them and no other."""
    N, C, H, W, F, R, S = shape
    dt = "f16"
    X, Wt = si.conv_inputs(N, C, H, W, F, R, S, dt, seed=94, dist="int")
    x, w = to_gpu(X, dt), to_gpu(Wt, dt)
    ref = torch.from_numpy(onum.conv2d(X, Wt, dt, (stride, stride), (1, 1), nthreads=16))
    touched = torch.zeros(ref.shape, dtype=torch.bool)
    for n, c, h, ww, v in ((0, 5, 0, 0, float("inf")), (N - 1, C - 1, H - 1, W - 1, float("nan")), (N // 2, 31, H // 2, 7, float("-inf"))):
        x[n, c, h, ww] = v
        for p in range(ref.shape[2]):
            for q in range(ref.shape[3]):
                if 0 <= h - (p * stride - 1) < R and 0 <= ww - (q * stride - 1) < S:
                    touched[n, :, p, q] = True
    Y = torch.zeros(ref.shape, dtype=torch.float32, device="cuda")
    nt.conv2d_implicit(x, w, Y, (stride, stride), (1, 1))
    torch.cuda.synchronize()
    assert nt.last_conv_plan().kernel == (nt.CONV_FEW_POSITIONS if H == 14 else nt.CONV_MANY_POSITIONS)
    y = Y.cpu().double()
    assert torch.equal(y[~touched], ref[~touched])
    assert not torch.isfinite(y[touched]).any()


def test_the_diagnostic_tells_the_kernels_of_a_path_apart():
    """Paths 6 and 7 stand for two kernels each; what ran otherwise, failed or was no convolution leaves nothing behind."""
    def run(shape, stride, tile=None, last=False):
        N, C, H, W, F, R, S = shape
        x, w = torch.zeros((N, C, H, W), dtype=torch.float16, device="cuda"), torch.zeros((F, C, R, S), dtype=torch.float16, device="cuda")
        if last:
            x = x.contiguous(memory_format=torch.channels_last)
        y = torch.empty((N, F, (H + 2 - R) // stride + 1, (W + 2 - S) // stride + 1), dtype=torch.float16, device="cuda")
        nt.conv2d_implicit(x, w, y, (stride, stride), (1, 1), tile=tile)
        torch.cuda.synchronize()
        p = nt.last_conv_plan()
        return nt.last_kernel_path(), p.kernel, p.filters, tuple(p.positions), tuple(p.tiles), p.wavefronts, p.runs
    nothing = (0, 0, (0, 0), (0, 0), 0, 0)
    assert run((2, 64, 14, 14, 64, 3, 3), 1)[:2] == (nt.PATH_CONV_CL, nt.CONV_FEW_POSITIONS)
    assert run((2, 64, 14, 14, 64, 3, 3), 1, last=True) == (nt.PATH_CONV_CL,) + nothing
    assert run((9, 64, 48, 48, 130, 3, 3), 1) == (nt.PATH_CONV_TAP, nt.CONV_MANY_POSITIONS, 256, (128, 96), (0, 216), 4, 2)
    assert run((9, 64, 48, 48, 130, 3, 3), 1, tile=(256, 256, 64)) == (nt.PATH_CONV_TAP,) + nothing
    assert run((30, 32, 56, 56, 160, 3, 3), 2)[:2] == (nt.PATH_CONV_CL, nt.CONV_MANY_POSITIONS)
    a = torch.zeros((64, 64), dtype=torch.float16, device="cuda")
    nt.gemm(a, a, torch.empty_like(a))
    assert nt.last_conv_plan().kernel == 0
    run((2, 64, 14, 14, 64, 3, 3), 1)
    with pytest.raises(nt.NtError):
        nt.gemm(a, a[:32], torch.empty_like(a))
    assert nt.last_conv_plan().kernel == 0
