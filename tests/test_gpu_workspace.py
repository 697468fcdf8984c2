"""GPU parity of the calls that go through the library's workspace when they overlap on one device, and of operands
whose last element a range-checked 16-byte load cannot fetch (odd pitches and extents, an operand that ends exactly at
the end of a page)."""
import threading

import numpy as np
import pytest
import torch

import paper_2507_11978_amd as nt
import synthetic_inputs as si
from oracle import numeric as onum
from gpu_util import TORCH_DT, to_f64, to_gpu

pytestmark = pytest.mark.gpu


def last(t):
    """the same tensor stored channels-last"""
    return t.contiguous(memory_format=torch.channels_last)


def test_two_streams_share_the_workspace_without_racing():
    """Two streams issue different k-split convolutions and skinny products at the same time, several rounds, no host
    synchronisation in between: each partial-tile region is handed from one call to the next through the library's
    event, so every result must be the exact integer result of its own problem."""
    dt = "f16"
    # (a) convolution, 12 programs x 72 k tiles -> split; (b) another one with other sizes (channels-last inputs: on the copy in the
    # workspace); (c), (d) skinny products
    Xa, Wa = si.conv_inputs(4, 512, 14, 14, 512, 3, 3, dt, seed=41, dist="int")
    Xb, Wb = si.conv_inputs(2, 256, 10, 10, 192, 3, 3, dt, seed=42, dist="int")
    Ac, Bc = si.gemm_inputs(16, 1024, 4096, dt, seed=43, dist="int")
    Ad, Bd = si.gemm_inputs(100, 520, 2048, dt, seed=44, dist="int")
    ref_a = onum.conv2d(Xa, Wa, dt, (1, 1), (0, 0), nthreads=16)
    ref_b = onum.conv2d(Xb, Wb, dt, (1, 1), (1, 1), nthreads=16)
    ref_c, ref_d = onum.gemm(Ac, Bc, dt), onum.gemm(Ad, Bd, dt)
    xa, wa, xb, wb = last(to_gpu(Xa, dt)), to_gpu(Wa, dt), last(to_gpu(Xb, dt)), to_gpu(Wb, dt)
    ac, bc, ad, bd = to_gpu(Ac, dt), to_gpu(Bc, dt), to_gpu(Ad, dt), to_gpu(Bd, dt)
    rounds = 6
    ya = [torch.full(ref_a.shape, float("nan"), dtype=torch.float32, device="cuda") for _ in range(rounds)]
    yb = [torch.full(ref_b.shape, float("nan"), dtype=torch.float32, device="cuda") for _ in range(rounds)]
    yc = [torch.full(ref_c.shape, float("nan"), dtype=torch.float32, device="cuda") for _ in range(rounds)]
    yd = [torch.full(ref_d.shape, float("nan"), dtype=torch.float32, device="cuda") for _ in range(rounds)]
    s1, s2 = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    for r in range(rounds):
        nt.conv2d_implicit(xa, wa, ya[r], (1, 1), (0, 0), stream=s1)
        assert nt.last_k_split() > 1 and nt.last_conv_plan().kernel == 0
        nt.gemm(ac, bc, yc[r], stream=s2)
        assert nt.last_k_split() > 1
        nt.conv2d_implicit(xb, wb, yb[r], (1, 1), (1, 1), stream=s2)
        assert nt.last_k_split() > 1 and nt.last_conv_plan().kernel == 0
        nt.gemm(ad, bd, yd[r], stream=s1)
        assert nt.last_k_split() > 1
    torch.cuda.synchronize()
    for r in range(rounds):
        assert np.array_equal(to_f64(ya[r]), ref_a), f"round {r}: convolution on stream 1"
        assert np.array_equal(to_f64(yb[r]), ref_b), f"round {r}: convolution on stream 2"
        assert np.array_equal(to_f64(yc[r]), ref_c), f"round {r}: product on stream 2"
        assert np.array_equal(to_f64(yd[r]), ref_d), f"round {r}: product on stream 1"


def test_two_streams_padded_copy_unfolded_and_channels_last_routes():
    """The same for the convolutions whose zero-padded copy, unfolded input or channels-last copy lives in the workspace: all
    three take turns on both streams."""
    dt, rounds = "f16", 6
    cases = []
    for seed, shape, stride, pad, path in [(51, (4, 16, 20, 20, 64, 5, 5), (1, 1), (2, 2), nt.PATH_CONV), (52, (4, 24, 21, 21, 64, 3, 3), (2, 2), (1, 1), nt.PATH_CONV_UNFOLD),
                                           (53, (4, 32, 21, 21, 64, 3, 3), (2, 2), (1, 1), nt.PATH_CONV_CL), (54, (4, 32, 20, 20, 64, 5, 5), (1, 1), (2, 2), nt.PATH_CONV_CL)]:
        X, Wt = si.conv_inputs(*shape, dt, seed=seed, dist="int")
        ref = onum.conv2d(X, Wt, dt, stride, pad, nthreads=16)
        ys = [torch.full(ref.shape, float("nan"), dtype=torch.float32, device="cuda") for _ in range(2 * rounds)]
        cases.append((last(to_gpu(X, dt)) if path == nt.PATH_CONV_CL else to_gpu(X, dt), to_gpu(Wt, dt), stride, pad, path, ref, ys))
    streams = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    for r in range(rounds):
        for i in range(len(cases)):
            for s in range(2):                                            # stream 0 at case i, stream 1 at the one after it
                x, w, stride, pad, path, _, ys = cases[(i + s) % len(cases)]
                nt.conv2d_implicit(x, w, ys[2 * r + s], stride, pad, stream=streams[s])
                assert nt.last_kernel_path() == path and nt.last_conv_plan().kernel == 0
    torch.cuda.synchronize()
    for _, _, stride, pad, path, ref, ys in cases:
        for r, y in enumerate(ys):
            assert np.array_equal(to_f64(y), ref), (r, path, stride)


def test_more_streams_than_parts_of_the_workspace():
    """Five streams, two threads: calls small enough for the workspace's small parts (a k split, a channels-last copy, a skinny
    product) meet on them and with calls that need the large one; every result is the exact one of its own problem."""
    dt, rounds = "f16", 5
    streams = [torch.cuda.Stream() for _ in range(5)]
    jobs = []
    for i in range(4):
        N, Cc, hw, K, stride = [(4, 256, 14, 256, 1), (2, 64, 30, 96, 2), (3, 128, 9, 70, 1), (1, 32, 57, 40, 2)][i]
        X, Wt = si.conv_inputs(N, Cc, hw, hw, K, 3, 3, dt, seed=60 + i, dist="int")
        ref = onum.conv2d(X, Wt, dt, (stride, stride), (1, 1), nthreads=16)
        x, w = last(to_gpu(X, dt)), to_gpu(Wt, dt)
        jobs.append((ref, lambda y, s, x=x, w=w, st=stride: nt.conv2d_implicit(x, w, y, (st, st), (1, 1), stream=s)))
    A, B = si.gemm_inputs(48, 640, 4096, dt, seed=65, dist="int")
    a, b = to_gpu(A, dt), to_gpu(B, dt)
    jobs.append((onum.gemm(A, B, dt), lambda y, s: nt.gemm(a, b, y, stream=s)))
    X, Wt = si.conv_inputs(16, 64, 112, 112, 32, 3, 3, dt, seed=66, dist="int")                      # a copy of 26 MB: with the filter's, and
    big_x, big_w = to_gpu(np.concatenate([X, X]), dt), to_gpu(Wt, dt)                                 # twice the images, more than a small part
    big_ref = onum.conv2d(X, Wt, dt, (2, 2), (1, 1), nthreads=16)
    jobs.append((np.concatenate([big_ref, big_ref]), lambda y, s: nt.conv2d_implicit(big_x, big_w, y, (2, 2), (1, 1), stream=s)))
    outs = [[torch.full(ref.shape, float("nan"), dtype=torch.float32, device="cuda") for ref, _ in jobs] for _ in range(2 * rounds)]
    torch.cuda.synchronize()

    def work(first):
        for r in range(first, 2 * rounds, 2):
            for j, (_, run) in enumerate(jobs):
                run(outs[r][j], streams[(r + j) % 5])
    threads = [threading.Thread(target=work, args=(i,)) for i in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    for r in range(2 * rounds):
        for j, (ref, _) in enumerate(jobs):
            assert np.array_equal(to_f64(outs[r][j]), ref), (r, j)


@pytest.mark.parametrize("warm", [False, True])
def test_calls_captured_into_a_graph(warm):
    """Strided and unit-stride convolutions and a split product captured on two streams of one capture, with and without calls
    on another stream before: replayed several times while the same calls run on that other stream, every result exact."""
    dt = "f16"
    jobs = []
    for i, (N, Cc, hw, K, stride) in enumerate([(2, 64, 30, 96, 2), (4, 256, 14, 256, 1), (8, 32, 28, 256, 1), (2, 48, 21, 40, 2)]):
        X, Wt = si.conv_inputs(N, Cc, hw, hw, K, 3, 3, dt, seed=70 + i, dist="int")
        ref = onum.conv2d(X, Wt, dt, (stride, stride), (1, 1), nthreads=16)
        jobs.append((ref, last(to_gpu(X, dt)) if i < 2 else to_gpu(X, dt), lambda x, y, s, w=to_gpu(Wt, dt), st=stride: nt.conv2d_implicit(x, w, y, (st, st), (1, 1), stream=s)))
    A, B = si.gemm_inputs(48, 640, 4096, dt, seed=75, dist="int")
    jobs.append((onum.gemm(A, B, dt), to_gpu(A, dt), lambda x, y, s, b=to_gpu(B, dt): nt.gemm(x, b, y, stream=s)))
    eager, main, side = torch.cuda.Stream(), torch.cuda.Stream(), torch.cuda.Stream()

    def outputs():
        return [torch.full(ref.shape, float("nan"), dtype=torch.float32, device="cuda") for ref, _, _ in jobs]
    loose = outputs()
    if warm:
        for (_, x, run), y in zip(jobs, loose):
            run(x, y, eager)
    torch.cuda.synchronize()
    captured, inputs = outputs(), [x.clone() for _, x, _ in jobs]
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=main):
        side.wait_stream(main)
        for j, ((_, _, run), x, y) in enumerate(zip(jobs, inputs, captured)):
            run(x, y, (main, side)[j % 2])
        main.wait_stream(side)
    for r in range(6):
        sign = 1.0 if r % 2 == 0 else -1.0                               # (other inputs each time: nothing left from the last replay)
        for (_, x, _), inp, y in zip(jobs, inputs, captured):
            torch.mul(x, sign, out=inp)
            y.fill_(float("nan"))
        for y in loose:
            y.fill_(float("nan"))
        torch.cuda.synchronize()
        with torch.cuda.stream(main):
            graph.replay()
        for (_, x, run), y in zip(jobs, loose):
            run(x, y, eager)
        torch.cuda.synchronize()
        for (ref, _, _), y, z in zip(jobs, captured, loose):
            assert np.array_equal(to_f64(y), sign * ref) and np.array_equal(to_f64(z), ref), r


def replay_two_at_once(run, problems, path_ok):
    """Each problem (operands, expected exact result) captured eight times over into a graph of its own; the graphs replayed at once
    on two streams, six rounds, every output compared."""
    graphs = []
    for args, want in problems:
        outs = [torch.full(want.shape, float("nan"), dtype=torch.float32, device="cuda") for _ in range(8)]
        stream, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
        torch.cuda.synchronize()
        with torch.cuda.graph(graph, stream=stream):
            for y in outs:
                run(*args, y, stream)
                assert path_ok(), nt.last_kernel_path()
        graphs.append((stream, graph, outs, want))
    for r in range(6):
        for _, _, outs, _ in graphs:
            for y in outs:
                y.fill_(float("nan"))
        torch.cuda.synchronize()
        for stream, graph, _, _ in graphs:
            with torch.cuda.stream(stream):
                graph.replay()
        torch.cuda.synchronize()
        for _, _, outs, want in graphs:
            for y in outs:
                assert np.array_equal(to_f64(y), want), r


@pytest.mark.parametrize("shape", [(18, 64, 48, 48, 72, 3, 3), (26, 32, 20, 20, 72, 3, 3), (16, 64, 56, 56, 72, 3, 2)])
def test_overlapping_replays_of_convolutions_that_need_no_workspace(shape):
    """Unit stride, at most 128 filters, many positions: an eager call may copy its filter into the workspace, a captured one must
    not, since nothing orders the replays of two graphs: two with filters of their own, replayed at once."""
    dt, pad = "f16", (1, 1)
    problems = []
    for seed in (80, 81):
        X, Wt = si.conv_inputs(*shape, dt, seed=seed, dist="int")
        problems.append(((to_gpu(X, dt), to_gpu(Wt, dt)), onum.conv2d(X, Wt, dt, (1, 1), pad, nthreads=16)))
    replay_two_at_once(lambda x, w, y, s: nt.conv2d_implicit(x, w, y, (1, 1), pad, stream=s), problems, lambda: nt.last_kernel_path() != nt.PATH_CONV_TAP)


@pytest.mark.parametrize("shape,stride,path", [((1, 8192, 7, 7, 64, 1, 1), 1, "PATH_DIRECT"), ((1, 2080, 13, 13, 300, 1, 1), 1, "PATH_CONV_DIRECT"),
                                               ((4, 384, 27, 27, 1000, 1, 1), 2, "PATH_CONV_UNFOLD")])
def test_overlapping_replays_of_convolutions_of_one_tap(shape, stride, path):
    """A very long reduction, one that a program's wavefronts share, a strided one: eager, the first and the last go through the workspace (a
    split, the unfolded input); captured, none does."""
    dt, problems = "f16", []
    for seed in (84, 85):
        X, Wt = si.conv_inputs(*shape, dt, seed=seed, dist="int")
        x, w = to_gpu(X, dt), to_gpu(Wt, dt)
        sub = x.float()[:, :, ::stride, ::stride]
        want = torch.matmul(w.float().reshape(shape[4], shape[1]), sub.reshape(shape[0], shape[1], -1)).reshape(shape[0], shape[4], *sub.shape[2:])
        problems.append(((x, w), want.double().cpu().numpy()))
    uses_it = lambda: nt.last_kernel_path() == nt.PATH_CONV_UNFOLD and nt.last_conv_plan().kernel == 0 or nt.last_kernel_path() == nt.PATH_CONV_DIRECT and nt.last_conv_plan().kernel == 0
    nt.conv2d_implicit(*problems[0][0], torch.empty(problems[0][1].shape, dtype=torch.float32, device="cuda"), (stride, stride))
    assert uses_it() == (shape[1] != 2080)
    replay_two_at_once(lambda x, w, y, s: nt.conv2d_implicit(x, w, y, (stride, stride), stream=s), problems,
                       lambda: nt.last_kernel_path() == getattr(nt, path) and not uses_it())


@pytest.mark.parametrize("product", [nt.gemm, nt.gemm_noalloc])
def test_overlapping_replays_of_products_with_a_ragged_k(product):
    """K no multiple of 64: split through scratch memory in an eager call, which captured ones -- two graphs replayed at once -- must
    leave alone."""
    dt, problems = "bf16", []
    for seed in (82, 83):
        A, B = si.gemm_inputs(48, 1500, 5408, dt, seed=seed, dist="int")
        problems.append(((to_gpu(A, dt), to_gpu(B, dt)), onum.gemm(A, B, dt)))
    (a, b), want = problems[0]
    y = torch.full(want.shape, float("nan"), dtype=torch.float32, device="cuda")
    product(a, b, y)
    torch.cuda.synchronize()
    assert nt.last_k_split() > 1 and np.array_equal(to_f64(y), want)
    replay_two_at_once(lambda a, b, y, s: product(a, b, y, stream=s), problems, lambda: nt.last_k_split() == 1)


@pytest.mark.parametrize("ta,tb", [(False, False), (False, True), (True, False), (True, True)])
@pytest.mark.parametrize("M,N,K", [(257, 259, 131), (300, 129, 97), (129, 131, 33), (255, 255, 31)])
def test_operand_that_ends_at_the_end_of_a_page(M, N, K, ta, tb):
    """Odd pitches and extents: the 4-byte word that holds an operand's last element would end 2 bytes past it, so a
    range-checked load drops it and the kernel fetches that element by itself.  Each operand is placed so that it
    ends exactly where a 4 KB page ends (NaNs follow where the allocation goes on); small integers: bit exact."""
    dt = "bf16"
    A, B = si.gemm_inputs(M, N, K, dt, seed=7 * M + K, dist="int")
    ref = onum.gemm(A, B, dt)

    def at_page_end(X, transposed):
        X = X.T.copy() if transposed else X
        buf = torch.full((X.size + 4096,), float("nan"), dtype=TORCH_DT[dt], device="cuda")
        end = (buf.data_ptr() + 2 * X.size + 4095) // 4096 * 4096            # first page end at or after the data's size
        first = (end - buf.data_ptr()) // 2 - X.size
        v = buf[first:first + X.size]
        v.copy_(to_gpu(X, dt).reshape(-1))
        assert (v.data_ptr() + 2 * X.size) % 4096 == 0
        v = v.view(X.shape)
        return v.t() if transposed else v

    for tile in [(128, 128, 64), (256, 256, 64)]:
        C = torch.full((M, N), float("nan"), dtype=torch.float32, device="cuda")
        nt.gemm(at_page_end(A, ta), at_page_end(B, tb), C, tile=tile)
        torch.cuda.synchronize()
        assert nt.last_kernel_path() == nt.PATH_DIRECT
        assert np.array_equal(to_f64(C), ref), (tile, ta, tb)


def test_zero_fill_of_many_batch_entries():
    """K = 0 zero-fills C; the batch may exceed what one grid dimension holds."""
    Bn, M, N = 70000, 3, 5
    A = torch.empty((Bn, M, 0), dtype=torch.float16, device="cuda")
    B = torch.empty((Bn, 0, N), dtype=torch.float16, device="cuda")
    C = torch.full((Bn, M, N), float("nan"), dtype=torch.float16, device="cuda")
    nt.bmm(A, B, C)
    torch.cuda.synchronize()
    assert (C == 0).all()
