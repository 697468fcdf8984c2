"""Convolutions that run in one launch straight from the caller's tensors (gemm_conv_patch.hip): 9 or 25 taps, or one and a stride, dense
planes, channels in whole blocks of 32, few positions or filters.  Small integers: every sum is exact, so the result must be the
oracle's bit for bit whatever the tile, the number of wavefronts that share the reduction and the patch's geometry."""
import numpy as np
import pytest
import torch

import paper_2507_11978_amd as nt
import synthetic_inputs as si
from oracle import numeric as onum
from gpu_util import TORCH_DT, inside, to_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,stride,pad,tile", [(*c, None) if len(c) == 3 else c for c in [
    # one shape for each kernel that is built: filters and positions per tile, wavefronts that share the reduction
    ((1, 64, 6, 6, 40, 3, 3), (2, 2), (1, 1), (16, 32, 2)),
    ((7, 128, 25, 25, 100, 3, 3), (2, 2), (1, 1), (16, 48, 4)),
    ((13, 96, 28, 28, 40, 3, 3), (1, 1), (1, 1), (16, 96, 3)),
    ((10, 128, 21, 21, 100, 3, 3), (2, 2), (1, 1), (32, 32, 4)),
    ((12, 64, 25, 25, 72, 3, 3), (1, 1), (1, 1), (32, 48, 2)),
    ((13, 64, 21, 21, 130, 3, 3), (1, 1), (1, 1), (32, 64, 2)),
    ((11, 96, 28, 28, 300, 3, 3), (2, 2), (1, 1), (32, 96, 3)),
    ((3, 96, 21, 21, 300, 3, 3), (1, 1), (1, 1), (64, 32, 3)),
    ((1, 64, 6, 6, 40, 5, 5), (2, 2), (2, 2), (16, 32, 2)),         # 25 taps
    ((7, 64, 21, 21, 40, 5, 5), (1, 1), (2, 2), (16, 64, 2)),
    ((7, 96, 28, 28, 40, 5, 5), (1, 1), (2, 2), (16, 96, 3)),
    ((1, 64, 14, 14, 40, 1, 1), (2, 2), (0, 0), (16, 32, 2)),       # one tap
    ((4, 352, 27, 27, 300, 1, 1), (2, 2), (0, 0), (32, 32, 6)),
    ((20, 64, 28, 28, 70, 1, 1), (2, 2), (0, 0)), ((9, 96, 56, 56, 130, 1, 1), (2, 2), (0, 0)), ((16, 96, 27, 25, 66, 1, 1), (2, 2), (0, 0)),
    ((2, 64, 9, 13, 24, 1, 1), (3, 1), (0, 0)), ((3, 64, 8, 9, 17, 1, 1), (1, 2), (2, 3)),
    ((2, 480, 7, 7, 103, 1, 1), (1, 1), (0, 0)), ((5, 512, 8, 9, 256, 1, 1), (1, 1), (0, 0)),      # ... unit stride, a reduction worth sharing
    ((8, 416, 13, 13, 88, 3, 3), (1, 1), (1, 1)), ((1, 480, 28, 28, 208, 5, 5), (1, 1), (2, 2)),   # long walks, one to two programs to a unit
    # edges of the patch
    ((4, 512, 14, 14, 512, 3, 3), (1, 1), (0, 0)),     # no padding, rows of 12: a tile's rows end at other places than the input's
    ((9, 96, 5, 5, 33, 3, 3), (1, 1), (1, 1)),         # 25 positions per image, odd planes: several images in a tile, 2-byte aligned runs
    ((40, 64, 2, 4, 17, 3, 3), (1, 1), (1, 1)),        # images of two runs
    ((1, 64, 1, 8, 8, 3, 3), (1, 1), (1, 1)),          # eight positions in all, rows of padding on both sides
    ((2, 288, 3, 50, 20, 3, 3), (1, 1), (1, 1)),       # nine blocks of channels (uneven shares), rows longer than a tile
    ((3, 64, 10, 9, 24, 9, 1), (1, 1), (4, 0)),        # nine taps in a column
    ((3, 64, 9, 13, 24, 1, 9), (2, 1), (0, 4)),        # ... in a row, mixed strides
    ((3, 160, 11, 7, 30, 3, 3), (3, 3), (2, 2)),       # stride as long as the filter, wide padding
    ((5, 64, 9, 8, 40, 3, 3), (4, 5), (0, 0)),         # rows and columns between the positions that no tap reads
    ((2, 64, 4, 6, 40, 5, 5), (1, 1), (4, 4)),         # more padding than image under some taps
]])
def test_conv_patch(shape, stride, pad, tile):
    N, C, H, W, F, R, S = shape
    for dt, out, lead in (("f16", "f32", 32), ("bf16", "bf16", 33), ("f16", "f16", 47)):
        X, Wt = si.conv_inputs(N, C, H, W, F, R, S, dt, seed=91, dist="int")
        ref = onum.conv2d(X, Wt, dt, stride, pad, nthreads=16)
        want = torch.from_numpy(ref).to(torch.float32).to(TORCH_DT[out])
        x, w = inside(to_gpu(X, dt), lead), inside(to_gpu(Wt, dt), 32)            # (rows of the filter stay 16-byte aligned)
        big = torch.full((N, F + 3, ref.shape[2], ref.shape[3]), float("nan"), dtype=TORCH_DT[out], device="cuda")
        Y = big[:, 2:F + 2]
        nt.conv2d_implicit(x, w, Y, stride, pad)
        torch.cuda.synchronize()
        plan = nt.last_conv_plan()
        path = nt.PATH_CONV_CL if R * S > 1 else nt.PATH_CONV_UNFOLD if max(stride) > 1 else nt.PATH_CONV_DIRECT
        assert plan.kernel == nt.CONV_FEW_POSITIONS and nt.last_kernel_path() == path and nt.last_k_split() == plan.wavefronts
        assert tile in (None, (plan.filters, plan.positions[0], plan.wavefronts))
        assert torch.equal(Y.cpu(), want), (shape, stride, pad, dt, out)
        assert torch.isnan(big[:, :2]).all() and torch.isnan(big[:, F + 2:]).all()


def test_conv_patch_of_a_channel_slice():
    """Images and channels further apart than their sizes, filters longer than the channels they are used with."""
    dt, N, C, H, W, F = "f16", 3, 96, 12, 11, 48
    X, Wt = si.conv_inputs(N, C + 64, H, W, F, 3, 3, dt, seed=92, dist="int")
    Xs, Ws = np.ascontiguousarray(X[:, 32:32 + C]), np.ascontiguousarray(Wt[:, 32:32 + C])
    ref = onum.conv2d(Xs, Ws, dt, (1, 1), (1, 1), nthreads=16)
    Y = torch.full(ref.shape, float("nan"), dtype=torch.float32, device="cuda")
    nt.conv2d_implicit(to_gpu(X, dt)[:, 32:32 + C], to_gpu(Wt, dt)[:, 32:32 + C], Y, (1, 1), (1, 1))
    torch.cuda.synchronize()
    assert nt.last_conv_plan().kernel == nt.CONV_FEW_POSITIONS
    assert np.array_equal(Y.double().cpu().numpy(), ref)


@pytest.mark.parametrize("shape", [(22, 448, 13, 13, 448), (2, 416, 7, 7, 103), (7, 128, 28, 28, 272), (2, 64, 56, 56, 383), (1, 32, 2, 4, 8), (300, 32, 3, 3, 40)])
def test_one_tap_of_unit_stride_is_a_product_per_image(shape):
    """However many positions, filters and images, of a slice of the channels."""
    N, C, H, W, F = shape
    dt = "f16"
    X, Wt = si.conv_inputs(N, C + 32, H, W, F, 1, 1, dt, seed=93, dist="int")
    ref = onum.conv2d(np.ascontiguousarray(X[:, 32:]), np.ascontiguousarray(Wt[:, 32:]), dt, (1, 1), (0, 0), nthreads=16)
    x, w = to_gpu(X, dt)[:, 32:], to_gpu(Wt, dt)[:, 32:]
    Y = torch.full(ref.shape, float("nan"), dtype=torch.float32, device="cuda")
    nt.conv2d_implicit(x, w, Y)
    torch.cuda.synchronize()
    assert nt.last_kernel_path() == nt.PATH_DIRECT and nt.last_k_split() == 1 and nt.last_conv_plan().kernel == 0
    assert np.array_equal(Y.double().cpu().numpy(), ref)


@pytest.mark.parametrize("shape", [(286, 96, 8, 8, 438), (260, 64, 8, 8, 500), (100, 64, 56, 56, 18)])
def test_one_tap_of_many_small_images_keeps_the_implicit_product(shape):
    """A product per image rounds each image's positions up to a tile: 12.5 / 15.3 us for the first of these."""
    N, C, H, W, F = shape
    X, Wt = si.conv_inputs(N, C, H, W, F, 1, 1, "f16", seed=94, dist="int")
    x, w = to_gpu(X, "f16"), to_gpu(Wt, "f16")
    Y = torch.full((N, F, H, W), float("nan"), dtype=torch.float32, device="cuda")
    nt.conv2d_implicit(x, w, Y)
    torch.cuda.synchronize()
    assert nt.last_kernel_path() == nt.PATH_CONV_DIRECT and nt.last_k_split() == 1 and nt.last_conv_plan().kernel == 0
    # (sums of small integers: exact in fp32 whatever their order)
    assert torch.equal(Y, torch.matmul(w.float().reshape(F, C), x.float().reshape(N, C, H * W)).reshape(Y.shape))


@pytest.mark.parametrize("shape", [(4, 384, 27, 27, 1000), (6, 608, 28, 28, 271)])
def test_one_strided_tap_is_unfolded_where_that_is_ahead(shape):
    """11.1 us for 13.0 straight from the caller's tensors, 12.6 for 15.3."""
    N, C, H, W, F = shape
    X, Wt = si.conv_inputs(N, C, H, W, F, 1, 1, "f16", seed=95, dist="int")
    x, w = to_gpu(X, "f16"), to_gpu(Wt, "f16")
    P, Q = (H + 1) // 2, (W + 1) // 2
    Y = torch.full((N, F, P, Q), float("nan"), dtype=torch.float32, device="cuda")
    nt.conv2d_implicit(x, w, Y, (2, 2))
    torch.cuda.synchronize()
    assert nt.last_kernel_path() == nt.PATH_CONV_UNFOLD and nt.last_conv_plan().kernel == 0
    sub = x.float()[:, :, ::2, ::2].reshape(N, C, P * Q)
    assert torch.equal(Y, torch.matmul(w.float().reshape(F, C), sub).reshape(Y.shape))


@pytest.mark.parametrize("shape,parts", [((1, 8192, 7, 7, 64), 32), ((1, 8192, 14, 14, 128), 32), ((3, 7200, 13, 13, 55), 23)])
def test_one_tap_of_a_very_long_reduction_stays_split(shape, parts):
    """As a product per image the whole reduction runs on a handful of programs: 30.0 us for 16.2, 38.5 for 21.0, 32.8 for 17.8."""
    N, C, H, W, F = shape
    X, Wt = si.conv_inputs(N, C, H, W, F, 1, 1, "f16", seed=96, dist="int")
    x, w = to_gpu(X, "f16"), to_gpu(Wt, "f16")
    Y = torch.full((N, F, H, W), float("nan"), dtype=torch.float32, device="cuda")
    nt.conv2d_implicit(x, w, Y)
    torch.cuda.synchronize()
    assert nt.last_kernel_path() == nt.PATH_CONV_DIRECT and nt.last_k_split() == parts and nt.last_conv_plan().kernel == 0
    assert torch.equal(Y, torch.matmul(w.float().reshape(F, C), x.float().reshape(N, C, H * W)).reshape(Y.shape))
