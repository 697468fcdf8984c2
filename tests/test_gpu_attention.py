"""GPU parity of nt_sdpa against the fp64 oracle (plain definition of attention).

Gates: the GEMM gates of this repository (max |err| <= 2e-2, relative Frobenius error <= 1e-2): the
probabilities are rounded to the 16-bit input format before they multiply V (as in the
FlashAttention-2 scheme), which bounds the relative error of an output by about one unit in the
last place of that format, and the output is rounded once more."""
import numpy as np
import pytest
import torch

import paper_2507_11978_amd as nt
import synthetic_inputs as si
from oracle import attention as oat
from oracle import numeric as onum
from gpu_util import TORCH_DT, assert_gates, to_f64, to_gpu

pytestmark = pytest.mark.gpu


def run(q, k, v, dt, scale=0.0):
    out = torch.full(q.shape[:-1] + (v.shape[-1],), float("nan"), dtype=TORCH_DT[dt], device="cuda")
    nt.sdpa(to_gpu(q, dt), to_gpu(k, dt), to_gpu(v, dt), out, scale=scale)
    torch.cuda.synchronize()
    return to_f64(out)


@pytest.mark.parametrize("dt", ["f16", "bf16"])
@pytest.mark.parametrize("B,H,Sq,Sk", [(1, 1, 128, 64), (2, 3, 256, 192), (1, 2, 100, 77), (1, 1, 1, 1), (2, 2, 33, 300), (1, 4, 384, 1024)])
def test_sdpa_shapes(dt, B, H, Sq, Sk):
    q, k, v = (si.normal_bits(s, dt, 10 + i, 1.0) for i, s in enumerate([(B, H, Sq, 64), (B, H, Sk, 64), (B, H, Sk, 64)]))
    ref = oat.sdpa(q, k, v, dt)
    assert_gates(run(q, k, v, dt), ref, dt, f"sdpa {dt} {B}x{H}x{Sq}x{Sk}")


def test_sdpa_closed_forms_and_scale():
    dt = "f16"
    rng = np.random.default_rng(2)
    v = si.round_to_bits(rng.integers(-4, 5, (1, 1, 200, 64)).astype(np.float32), dt)
    k = si.normal_bits((1, 1, 200, 64), dt, 3, 1.0)
    # zero queries: the mean of the values (exact up to the rounding of the weights 1/200 and of the result)
    got = run(np.zeros((1, 1, 70, 64), dtype=np.uint16), k, v, dt)
    assert np.abs(got - onum.decode(v, dt).mean(axis=2, keepdims=True)).max() < 4e-3
    # a dominant key takes all the weight: its value row comes out exactly
    q = si.normal_bits((1, 1, 5, 64), dt, 4, 1.0)
    kd = onum.decode(k, dt).copy()
    kd[0, 0, 17] = onum.decode(q, dt)[0, 0, 2] * 8.0
    k2 = si.round_to_bits(kd.astype(np.float32), dt)
    got = run(q, k2, v, dt, scale=1.0)
    assert np.array_equal(got[0, 0, 2], onum.decode(v, dt)[0, 0, 17])
    # an explicit scale against the oracle; large scores must not overflow
    q, k, v = (si.normal_bits((1, 2, 130, 64), dt, 20 + i, 3.0) for i in range(3))
    assert_gates(run(q, k, v, dt, scale=0.5), oat.sdpa(q, k, v, dt, scale=0.5), dt, "sdpa scale 0.5")


def test_sdpa_strided_views_and_errors():
    dt, B, H, S = "f16", 2, 3, 150
    q, k, v = (si.normal_bits((B, H, S, 64), dt, 30 + i, 1.0) for i in range(3))
    ref = oat.sdpa(q, k, v, dt)
    # [batch, seq, heads, 64] storage viewed as [batch, heads, seq, 64]; output into a padded buffer
    qs = to_gpu(np.ascontiguousarray(q.transpose(0, 2, 1, 3)), dt).permute(0, 2, 1, 3)
    ks = to_gpu(np.ascontiguousarray(k.transpose(0, 2, 1, 3)), dt).permute(0, 2, 1, 3)
    vbuf = torch.zeros((B, H, S, 80), dtype=torch.float16, device="cuda")
    vbuf[..., :64] = to_gpu(v, dt)
    obuf = torch.full((B, H, S + 2, 64), -7.0, dtype=torch.float16, device="cuda")
    nt.sdpa(qs, ks, vbuf[..., :64], obuf[:, :, 1:S + 1])
    torch.cuda.synchronize()
    assert_gates(to_f64(obuf[:, :, 1:S + 1]), ref, dt, "sdpa strided")
    assert (obuf[:, :, 0] == -7.0).all() and (obuf[:, :, S + 1] == -7.0).all()
    z = torch.zeros((1, 1, 8, 32), dtype=torch.float16, device="cuda")
    with pytest.raises(nt.NtError):
        nt.sdpa(z, z, z, z)                                               # head size 32 is not built
    a = torch.zeros((1, 1, 8, 64), dtype=torch.float16, device="cuda")
    with pytest.raises(nt.NtError):
        nt.sdpa(a, a[:, :, :0], a[:, :, :0], a)                           # no keys
    with pytest.raises(nt.NtError):
        nt.sdpa(a, a, a[:, :, :4], a)                                     # K and V lengths differ


def test_sdpa_negative_scale():
    dt = "f16"
    q, k, v = (si.normal_bits((1, 2, 90, 64), dt, 40 + i, 1.0) for i in range(3))
    assert_gates(run(q, k, v, dt, scale=-0.3), oat.sdpa(q, k, v, dt, scale=-0.3), dt, "sdpa negative scale")


@pytest.mark.parametrize("dt", ["f16", "bf16"])
def test_sdpa_scores_rising_along_the_keys(dt):
    """Keys grow along the sequence, so a row's maximum keeps rising (or falling) from block to block: some
    blocks stay within the band the kernel tolerates between its row reference and the running maximum, others
    force the reference up."""
    rng = np.random.default_rng(70)
    S, Sk = 96, 640
    w = rng.standard_normal(64).astype(np.float32)
    w /= np.linalg.norm(w)
    for per_block in (3.0, 11.0, 40.0):                       # rise of the top score per 64 keys, in base-2 units
        q = rng.standard_normal((1, 2, S, 64)).astype(np.float32)
        proj = np.abs(q @ w).mean()
        step = per_block / 64.0 / (proj * 0.125 * 1.4427)      # so that scale * q . k_j grows by ~per_block per block
        kf = (np.arange(Sk, dtype=np.float32)[:, None] * step) * w[None, :] + 0.05 * rng.standard_normal((Sk, 64)).astype(np.float32)
        kf = np.broadcast_to(kf, (1, 2, Sk, 64))
        qb, kb = si.round_to_bits(q, dt), si.round_to_bits(np.ascontiguousarray(kf), dt)
        vb = si.normal_bits((1, 2, Sk, 64), dt, 71, 1.0)
        assert_gates(run(qb, kb, vb, dt), oat.sdpa(qb, kb, vb, dt), dt, f"sdpa rising scores {per_block} {dt}")


@pytest.mark.parametrize("dt", ["f16", "bf16"])
@pytest.mark.parametrize("B,H,Sq,Sk", [(1, 1, 1, 1), (1, 3, 2, 7), (2, 5, 1, 8), (1, 9, 2, 31), (3, 3, 1, 33), (1, 1, 1, 511), (2, 8, 2, 513), (1, 17, 1, 1057),
                                       (1, 8, 32, 96), (1, 16, 16, 1030), (2, 96, 1, 70)])
def test_few_queries(dt, B, H, Sq, Sk):
    """A workgroup per query: fewer keys than lane groups, than wavefronts' batches, ragged last batches, several batches per
    wavefront, head counts that are and are not multiples of eight; scores that rise along the keys; strided operands."""
    q, k, v = (si.normal_bits(s, dt, 80 + i, 1.5) for i, s in enumerate([(B, H, Sq, 64), (B, H, Sk, 64), (B, H, Sk, 64)]))
    ref = oat.sdpa(q, k, v, dt)
    assert_gates(run(q, k, v, dt), ref, dt, f"sdpa {dt} {B}x{H}x{Sq}x{Sk}")
    kd = onum.decode(k, dt) * np.linspace(0.1, 6.0, Sk)[None, None, :, None]
    kb = si.round_to_bits(kd.astype(np.float32), dt)
    ref = oat.sdpa(q, kb, v, dt, scale=-0.4)
    qs, ks, vs = (to_gpu(np.ascontiguousarray(t.transpose(0, 2, 1, 3)), dt).permute(0, 2, 1, 3) for t in (q, kb, v))
    vbuf = torch.full((B, H, Sk + 1, 71), float("nan"), dtype=TORCH_DT[dt], device="cuda")       # rows of odd pitch, NaN behind the keys
    vbuf[:, :, :Sk, 3:67] = vs
    obuf = torch.full((B, H, Sq, 66), -7.0, dtype=TORCH_DT[dt], device="cuda")
    nt.sdpa(qs, ks, vbuf[:, :, :Sk, 3:67], obuf[..., 1:65], scale=-0.4)
    torch.cuda.synchronize()
    assert_gates(to_f64(obuf[..., 1:65]), ref, dt, f"sdpa strided {dt} {B}x{H}x{Sq}x{Sk}")
    assert (obuf[..., 0] == -7.0).all() and (obuf[..., 65] == -7.0).all()


@pytest.mark.parametrize("dt", ["f16", "bf16"])
@pytest.mark.parametrize("Sk", [1, 63, 64, 65, 128, 129, 192, 321, 705, 768, 833, 1025])
def test_key_blocks_of_every_kind_of_rows(dt, Sk):
    """One to seventeen key blocks (the rings hold three and two, twelve and more are dealt out to four groups of wavefronts), a last block of one key, of all but one; rows that the range-checked
    loads take -- dense, pitched, of odd pitch with NaN between and behind them -- and rows they do not (a key repeated for
    every position): the same result."""
    B, H, Sq = 1, 3, 130
    q, k, v = (si.normal_bits((B, H, n, 64), dt, 90 + i, 1.5) for i, n in enumerate([Sq, Sk, Sk]))
    ref = oat.sdpa(q, k, v, dt)
    gq, gk, gv = (to_gpu(t, dt) for t in (q, k, v))
    out = torch.full((B, H, Sq, 64), float("nan"), dtype=TORCH_DT[dt], device="cuda")
    nt.sdpa(gq, gk, gv, out)
    torch.cuda.synchronize()
    assert_gates(to_f64(out), ref, dt, f"sdpa {dt} {Sk} keys")
    for pitch, at in ((72, 8), (67, 1)):
        views = []
        for t in (gk, gv):
            buf = torch.full((B, H, Sk + 70, pitch), float("nan"), dtype=TORCH_DT[dt], device="cuda")
            buf[:, :, :Sk, at:at + 64] = t
            views.append(buf[:, :, :Sk, at:at + 64])
        o2 = torch.full_like(out, float("nan"))
        nt.sdpa(gq, views[0], views[1], o2)
        torch.cuda.synchronize()
        assert torch.equal(o2, out), pitch
    one_k, one_v = gk[:, :, :1].expand(B, H, Sk, 64), gv[:, :, :1].expand(B, H, Sk, 64)      # stride 0 along the keys
    o3 = torch.full_like(out, float("nan"))
    nt.sdpa(gq, one_k, one_v, o3)
    o4 = torch.full_like(out, float("nan"))
    nt.sdpa(gq, one_k.contiguous(), one_v.contiguous(), o4)
    torch.cuda.synchronize()
    assert torch.equal(o3, o4)


@pytest.mark.parametrize("dt", ["f16", "bf16"])
@pytest.mark.parametrize("Sk", [65, 321, 833])
def test_keys_spread_over_more_than_two_gigabytes(dt, Sk):
    """A pitch at which a head's keys reach past the range-checked loads' offsets: through registers, one group whatever the number
    of blocks; the same as from a copy of theirs (13 blocks of the copy are dealt out to groups)."""
    H, Sq, pitch = 3, 130, (1 << 30) // (Sk + 640) + 7                 # elements
    q, k, v = (to_gpu(si.normal_bits((1, H, n, 64), dt, 150 + i, 1.0), dt) for i, n in enumerate([Sq, Sk, Sk]))
    buf = torch.zeros(((Sk - 1) * pitch + 2 * H * 64,), dtype=TORCH_DT[dt], device="cuda")
    far = [buf[i * H * 64:].as_strided((1, H, Sk, 64), (0, 64, pitch, 1)) for i in range(2)]
    for dst, src in zip(far, (k, v)):
        dst.copy_(src)
    got, near, ref = (torch.full_like(q, float("nan")) for _ in range(3))
    nt.sdpa(q, far[0], far[1], got)
    nt.sdpa(q, far[0], v, near)
    nt.sdpa(q, k, v, ref)
    torch.cuda.synchronize()
    assert torch.equal(got, near)
    if Sk < 705:
        assert torch.equal(got, ref)
    assert_gates(to_f64(got), to_f64(ref), dt, f"sdpa keys of pitch {pitch}")


# how the keys are dealt out follows from the number of (head, query block) programs and of key blocks: four groups of one wavefront share
# them, with row sums on either pipe, two groups of four do, a workgroup per query, one group of four wavefronts, of eight (256 queries)
WALKS = [(2, 3, 130, 640), (1, 3, 130, 1024), (1, 3, 130, 1025), (1, 150, 130, 832), (1, 3, 1, 1024), (1, 129, 400, 700), (1, 128, 511, 640)]
LAYOUTS = [(32, 4, 4, 0), (32, 4, 4, 0), (32, 4, 4, 1), (128, 2, 8, 1), (1, 1, 16, 0), (128, 1, 4, 1), (256, 1, 8, 1)]


def layout():
    p = nt.last_sdpa_plan()
    return p.queries, p.groups, p.wavefronts, p.matrix_sums


@pytest.mark.parametrize("dt", ["f16", "bf16"])
@pytest.mark.parametrize("B,H,Sq,Sk,plan", [(*w, p) for w, p in zip(WALKS, LAYOUTS)])
def test_scores_of_minus_infinity(dt, B, H, Sq, Sk, plan):
    """Keys masked by a score of -inf (an infinite key channel; a lowest value whose product overflows) have weight 0 wherever
    they lie: whole key blocks of them first, last, all around, in some queries of a wavefront and not in others."""
    q, k, v = (onum.decode(si.normal_bits((B, H, n, 64), dt, 110 + i, 1.0), dt).astype(np.float32) for i, n in enumerate([Sq, Sk, Sk]))
    q[..., 0], k[..., 0] = 1.0, 0.0
    v = si.round_to_bits(v, dt)
    low = -65504.0 if dt == "f16" else -3.3895314e38
    for alive in (slice(0, 64), slice(Sk - 64, Sk), slice(Sk - 1, Sk), slice(300, 311), slice(64, 600)):
        masked = np.ones(Sk, dtype=bool)
        masked[alive] = False
        for mask, channel in ((-np.inf, 1.0), (low, 4.0 if dt == "bf16" else 65504.0)):
            qm, km = q.copy(), k.copy()
            qm[..., 0] = channel
            if mask == low:
                qm[..., ::2, 0] = 0.0                                # every other query sees all keys
            km[..., masked, 0] = mask
            qb, kb = si.round_to_bits(qm, dt), si.round_to_bits(km, dt)
            heads = slice(0, 3 if H > 100 and Sq > 130 else H)       # (the oracle's time)
            ref, got = oat.sdpa(qb[:, heads], kb[:, heads], v[:, heads], dt), run(qb, kb, v, dt)
            assert layout() == plan and np.isfinite(got).all()
            assert_gates(got[:, heads], ref, dt, f"sdpa {dt} {B}x{H}x{Sq}x{Sk} alive {alive} mask {mask}")
    k[..., 0] = -np.inf                                              # no key at all: 0 / 0, as in the definition
    assert np.isnan(run(si.round_to_bits(q, dt), si.round_to_bits(k, dt), v, dt)).all()


@pytest.mark.parametrize("dt", ["f16", "bf16"])
@pytest.mark.parametrize("Sk", [1, 64, 65, 129, 705])
@pytest.mark.parametrize("H", [3, 150])
def test_rows_that_overlap(dt, H, Sk):
    """Keys and values whose rows overlap (pitch 63, 40, 0: not for the range-checked loads): the same bits as from a copy of
    theirs, one block, blocks ahead of each other, a last block of one key; and with enough keys for groups."""
    Sq = 130
    gq = to_gpu(si.normal_bits((1, H, Sq, 64), dt, 130, 1.0), dt)
    for n in (Sk, Sk + 700):
        for pitch in (63, 40, 0):
            k, v = (to_gpu(si.normal_bits((H * n * pitch + 64,), dt, 131 + i, 1.0), dt).as_strided((1, H, n, 64), (0, n * pitch, pitch, 1)) for i in range(2))
            got, ref = torch.full_like(gq, float("nan")), torch.full_like(gq, float("nan"))
            nt.sdpa(gq, k, v, got)
            nt.sdpa(gq, k.contiguous(), v.contiguous(), ref)
            torch.cuda.synchronize()
            assert_gates(to_f64(ref), oat.sdpa(*(t.contiguous().cpu().view(torch.int16).numpy().view(np.uint16) for t in (gq, k, v)), dt), dt, f"sdpa {n}")
            if H == 3 or n < 705:
                assert torch.equal(got, ref), (n, pitch)             # (300 programs: groups for the copy, none for these rows)
            assert_gates(to_f64(got), to_f64(ref), dt, f"sdpa rows of pitch {pitch}, {n} keys")


@pytest.mark.parametrize("dt", ["f16", "bf16"])
@pytest.mark.parametrize("B,H,Sq,Sk", [(1, 3, 130, 1393), (1, 150, 130, 833), (1, 257, 10, 770)])
def test_keys_dealt_to_groups_with_references_far_apart(dt, B, H, Sq, Sk):
    """Scores that rise (scale > 0) or fall (scale < 0) along the keys, slowly and by hundreds of powers of two from end to end:
    the groups of wavefronts that share the keys end with references far apart, and a group's last block may be missing."""
    rng = np.random.default_rng(120)
    w = rng.standard_normal(64).astype(np.float32)
    w /= np.linalg.norm(w)
    q = rng.standard_normal((B, H, Sq, 64)).astype(np.float32)
    q += (2.0 - q @ w)[..., None] * w                                # every query's component along w is 2
    vb = si.normal_bits((B, H, Sk, 64), dt, 121, 1.0)
    qb = si.round_to_bits(q, dt)
    for per_block in (2.0, 30.0):                                    # rise per 64 keys, in base-2 units
        step = per_block / 64.0 / (2.0 * 0.125 * 1.4427)
        kf = (np.arange(Sk, dtype=np.float32)[:, None] * step) * w[None, :] + 0.05 * rng.standard_normal((Sk, 64)).astype(np.float32)
        kb = si.round_to_bits(np.ascontiguousarray(np.broadcast_to(kf, (B, H, Sk, 64))), dt)
        for scale in (0.125, -0.125):
            assert_gates(run(qb, kb, vb, dt, scale=scale), oat.sdpa(qb, kb, vb, dt, scale=scale), dt, f"sdpa {dt} {H} heads {per_block} {scale}")


@pytest.mark.parametrize("Sq", [1, 3])
def test_more_heads_than_one_launch_holds(Sq):
    """2^24 + 32768 heads: with one key every query's result is its head's value row."""
    B, H = 513, 32768
    vc = (torch.arange(H, device="cuda") % 251).to(torch.bfloat16).reshape(1, H, 1, 1).expand(1, H, 1, 64).contiguous().expand(B, H, 1, 64)
    one = torch.zeros((1, 1, 1, 64), dtype=torch.bfloat16, device="cuda")
    out = torch.empty((B, H, Sq, 64), dtype=torch.bfloat16, device="cuda").fill_(float("nan"))
    nt.sdpa(one.expand(B, H, Sq, 64), one.expand(B, H, 1, 64), vc, out)
    torch.cuda.synchronize()
    assert all(torch.equal(out[b], vc[b].expand(H, Sq, 64)) for b in (0, 1, 510, 511, 512))


def test_few_queries_weigh_in_fp32():
    """One query per head: scores, weights and sums stay in fp32, so all but a few results are the fp64 result rounded once."""
    B, H, Sk = 2, 24, 2047
    q, k, v = (si.normal_bits((B, H, n, 64), "bf16", 140 + i, 1.0) for i, n in enumerate([1, Sk, Sk]))
    want = torch.from_numpy(oat.sdpa(q, k, v, "bf16")).to(torch.bfloat16)
    got = torch.from_numpy(run(q, k, v, "bf16")).to(torch.bfloat16)
    assert (got != want).float().mean() < 0.01                       # (a result within fp32 error of the middle between two)


@pytest.mark.parametrize("dt", ["f16", "bf16"])
@pytest.mark.parametrize("B,H,Sq,Sk", [
    # launches that leave units empty: blocks of 32 queries in one, two and four groups of one wavefront ...
    (1, 7, 33, 64), (2, 3, 97, 65), (1, 5, 160, 384), (1, 9, 64, 385), (2, 4, 129, 449), (1, 64, 128, 511), (1, 2, 1000, 1025),
    # ... of 64 in as many groups of two, up to a full round of the units ...
    (1, 65, 97, 33), (2, 16, 300, 70), (1, 64, 256, 700), (1, 51, 320, 705), (4, 16, 200, 769),
    # ... of 128: two groups from seven blocks of keys on, four from twelve
    (1, 129, 129, 400), (1, 128, 200, 449), (1, 128, 140, 705)])
def test_blocks_of_queries_of_every_width(dt, B, H, Sq, Sk):
    q, k, v = (si.normal_bits((B, H, n, 64), dt, 150 + i, 1.0) for i, n in enumerate([Sq, Sk, Sk]))
    ref = oat.sdpa(q, k, v, dt)
    assert_gates(run(q, k, v, dt), ref, dt, f"sdpa {dt} {B}x{H}x{Sq}x{Sk}")
    # rows of K and V that overlap go through registers: the same walk, the same bits as from a copy
    if Sq * H < 3000:
        gq = to_gpu(q, dt)
        gk, gv = (to_gpu(si.normal_bits((B * H * Sk * 60 + 64,), dt, 155 + i, 1.0), dt).as_strided((B, H, Sk, 64), (H * Sk * 60, Sk * 60, 60, 1)) for i in range(2))
        got, want = torch.full_like(gq, float("nan")), torch.full_like(gq, float("nan"))
        nt.sdpa(gq, gk, gv, got)
        nt.sdpa(gq, gk.contiguous(), gv.contiguous(), want)
        torch.cuda.synchronize()
        assert torch.equal(got, want)


@pytest.mark.parametrize("dt", ["f16", "bf16"])
@pytest.mark.parametrize("B,H,Sq,Sk,plan", [
    # groups with enough blocks to walk take their row sums on the matrix pipe: the first such number of blocks and the one before,
    # one wavefront a group in four groups, two in two, four in one, and that with more programs than are resident
    (1, 3, 64, 1024, (32, 4, 4, 0)), (1, 3, 64, 1025, (32, 4, 4, 1)), (1, 64, 256, 256, (64, 2, 4, 0)), (1, 64, 256, 257, (64, 2, 4, 1)), (1, 64, 256, 640, (64, 2, 4, 1)), (1, 64, 256, 641, (64, 2, 4, 1)),
    (1, 130, 400, 128, (128, 1, 4, 0)), (1, 130, 400, 129, (128, 1, 4, 1)), (5, 52, 512, 64, (128, 1, 4, 0)), (5, 52, 512, 65, (128, 1, 4, 1)), (5, 52, 512, 128, (128, 1, 4, 1)),
    # ... always: two wavefronts a group in four groups, four in two and in four
    (1, 64, 256, 705, (64, 4, 8, 1)), (1, 128, 200, 449, (128, 2, 8, 1)), (1, 128, 140, 705, (128, 4, 16, 1)),
    # ... never: two groups of one wavefront, one group of one and of two
    (2, 3, 97, 384, (32, 2, 2, 0)), (1, 7, 33, 64, (32, 1, 1, 0)), (1, 65, 97, 33, (64, 1, 2, 0)),
    # blocks of 256 queries: whole ones, a last one of one query and of all but one
    (1, 64, 1024, 129, (256, 1, 8, 1)), (1, 96, 1025, 150, (256, 1, 8, 1)), (1, 128, 511, 193, (256, 1, 8, 1)), (3, 43, 511, 193, (128, 1, 4, 1))])
def test_row_sums_of_walks_of_every_length(dt, B, H, Sq, Sk, plan):
    """Against the definition, with scores that raise the reference late; a query of NaN stays the only one."""
    q, k, v = (si.normal_bits((B, H, n, 64), dt, 160 + i, 1.0) for i, n in enumerate([Sq, Sk, Sk]))
    kd = onum.decode(k, dt).astype(np.float32)
    kd[:, :, -40:] *= 6.0
    k = si.round_to_bits(kd, dt)
    got = run(q, k, v, dt)
    assert layout() == plan
    heads = slice(0, 3)
    assert_gates(got[:, heads], oat.sdpa(q[:, heads], k[:, heads], v[:, heads], dt), dt, f"sdpa {dt} {B}x{H}x{Sq}x{Sk}")
    assert np.isfinite(got).all()
    holes = np.arange(5, Sq, 37)
    q[:, :, holes, 9] = 0x7e00 if dt == "f16" else 0x7fc0
    with_nan = run(q, k, v, dt)
    assert np.isnan(with_nan[:, :, holes]).all()
    rest = np.delete(np.arange(Sq), holes)
    # (a wavefront that holds a NaN sets its reference anew for every block: the others' results move by their weights' rounding, within the gates)
    assert_gates(with_nan[:, heads][:, :, rest], got[:, heads][:, :, rest], dt, "sdpa beside NaN")


@pytest.mark.parametrize("dt", ["f16", "bf16"])
@pytest.mark.parametrize("H,Sk,waves", [(160, 256, 4), (160, 257, 8), (160, 640, 8), (161, 640, 4), (160, 641, 16), (256, 641, 16), (257, 641, 4), (512, 385, 4), (513, 384, 4), (513, 385, 8)])
def test_one_query_on_every_number_of_wavefronts(dt, H, Sk, waves):
    q, k, v = (si.normal_bits((1, H, n, 64), dt, 170 + i, 1.5) for i, n in enumerate([1, Sk, Sk]))
    assert_gates(run(q, k, v, dt), oat.sdpa(q, k, v, dt), dt, f"sdpa {dt} {H} heads x {Sk}")
    assert layout() == (1, 1, waves, 0)
