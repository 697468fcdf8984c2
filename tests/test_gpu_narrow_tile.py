"""The 64 x 64 tile, whose loop takes two 32-k slices per trip out of a ring of eight: every number of slices up to a few rings, odd
numbers of them and of pairs, ragged ends; aligned and unaligned rows, both layouts of B.  Small integers: bit for bit."""
import numpy as np
import pytest
import torch

import paper_2507_11978_amd as nt
import synthetic_inputs as si
from oracle import numeric as onum
from gpu_util import to_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K", [1, 8, 31, 32, 33, 64, 65, 96, 97, 128, 129, 191, 192, 224, 255, 256, 257, 288, 320, 351, 511, 512, 513, 577, 640, 703])
@pytest.mark.parametrize("M,N", [(64, 64), (70, 130)])
def test_every_number_of_slices(M, N, K):
    for dt, bt, pitch in (("f16", False, 0), ("bf16", True, 0), ("f16", True, 3)):
        A, B = si.gemm_inputs(M, N, K, dt, seed=K, dist="int")
        ref = onum.gemm(A, B, dt)
        a, b = to_gpu(A, dt), to_gpu(np.ascontiguousarray(B.T) if bt else B, dt)
        if pitch:                                             # rows further apart than they are long, NaN between them
            wide = [torch.full((t.shape[0], t.shape[1] + pitch), float("nan"), dtype=t.dtype, device="cuda") for t in (a, b)]
            for w, t in zip(wide, (a, b)):
                w[:, :t.shape[1]] = t
            a, b = (w[:, :w.shape[1] - pitch] for w in wide)
        C = torch.full((M, N), float("nan"), dtype=torch.float32, device="cuda")
        nt.gemm(a, b.t() if bt else b, C, tile=(64, 64, 32))
        torch.cuda.synchronize()
        assert K < 8 or nt.last_kernel_path() == nt.PATH_DIRECT
        assert np.array_equal(C.double().cpu().numpy(), ref), (M, N, K, dt, bt, pitch)
