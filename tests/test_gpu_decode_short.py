"""Decode steps over few, short rows: whole rows in one workgroup up to a length, sliced rows behind it; and the
device-counted step, which issues its first loads before it knows the new token's slot: the slot wanders through every
block of the row here."""
import numpy as np
import pytest

import synth
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu
BF16, F32 = synth.BF16, synth.F32


@pytest.mark.parametrize("Hq,Hkv,d", [(8, 2, 128), (4, 2, 64), (7, 1, 128), (12, 1, 64)])
@pytest.mark.parametrize("dtype,n", [(BF16, 1), (BF16, 33), (BF16, 128), (BF16, 129), (BF16, 255), (BF16, 256), (BF16, 257), (BF16, 600),
                                     (F32, 1), (F32, 127), (F32, 128), (F32, 129), (F32, 256), (F32, 257), (F32, 600)])
@pytest.mark.parametrize("ring", [False, True])
def test_steps_around_the_single_pass_length(ref, dtype, n, Hq, Hkv, d, ring):
    import torch

    import paper_2503_08879_amd as sk

    P = 2
    W = n  # the whole row is the window: the slot takes every position
    rng = np.random.default_rng(n * 31 + Hq + d)
    draw = lambda *shape: synth.round_to_dtype(rng.standard_normal(shape, dtype=np.float32), dtype)
    Kc, Vc = draw(P, Hkv, n, d), draw(P, Hkv, n, d)
    Kd, Vd = synth.host_to_torch(Kc, dtype), synth.host_to_torch(Vc, dtype)
    desc, ws, out = gu.gpu_decode_setup(dtype, P, Hq, Hkv, d, 0, 0, W, n)
    state = torch.zeros(2, dtype=torch.int32, device="cuda")
    # a few steps at spread positions of the window, wrap-around included
    for t in sorted({0, 1, n // 3, n - 1, n, n + n // 2}):
        q, kn, vn = draw(P, Hq, d), draw(P, Hkv, d), draw(P, Hkv, d)
        Kc[:, :, t % W], Vc[:, :, t % W] = kn, vn
        want = ref.decode_attn(dtype, 0, q, Kc, Vc, n)
        ins = [synth.host_to_torch(x, dtype) for x in (q, kn, vn)]
        if ring:
            state[0] = t
            sk.sagekv_decode_step_ring(desc, *ins, Kd, Vd, state, out, ws)
            assert state.tolist() == [t + 1, 0]
        else:
            sk.sagekv_decode_step(desc, *ins, Kd, Vd, t, out, ws)
        # up to 128 tokens and 4 heads the weights stay fp32: sums of up to 128 products of order 1, fp32 logits
        atol = 1e-5 if dtype == BF16 and n <= 128 and Hq // Hkv <= 4 else gu.DECODE_ATOL[dtype]
        assert np.abs(out.cpu().numpy() - want).max() <= atol, t
        np.testing.assert_array_equal(synth.torch_to_host(Kd, dtype), Kc)
        np.testing.assert_array_equal(synth.torch_to_host(Vd, dtype), Vc)


@pytest.mark.parametrize("Hq,Hkv,d", [(8, 2, 128), (7, 1, 64), (12, 1, 128)])
@pytest.mark.parametrize("n,slot", [(45, 0), (100, 0), (200, 0), (200, 192), (601, 0), (601, 512), (601, 592)])
@pytest.mark.parametrize("paged", [False, True])
def test_a_non_finite_token_leaves_with_the_step_that_replaces_it(ref, n, slot, Hq, Hkv, d, paged):
    """The device-counted step reads its first blocks before it knows the slot, and lanes past a ragged end read the first
    token of their slice (pages: of their group of 16) instead: where that token is the one being replaced, its old
    value must not reach the sums, not even with weight 0."""
    import torch

    import paper_2503_08879_amd as sk

    P, page = 2, 16
    rng = np.random.default_rng(n + slot + Hq)
    draw = lambda *shape: synth.round_to_dtype(rng.standard_normal(shape, dtype=np.float32), BF16)
    Kc, Vc, q, kn, vn = draw(P, Hkv, n, d), draw(P, Hkv, n, d), draw(P, Hq, d), draw(P, Hkv, d), draw(P, Hkv, d)
    Kd, Vd = synth.host_to_torch(Kc, BF16), synth.host_to_torch(Vc, BF16)
    Kd[:, :, slot] = float("nan")
    Vd[:, :, slot] = float("inf")
    Kc[:, :, slot], Vc[:, :, slot] = kn, vn
    want = ref.decode_attn(BF16, 0, q, Kc, Vc, n)
    desc, ws, out = gu.gpu_decode_setup(BF16, P, Hq, Hkv, d, 0, 0, n, n)
    state = torch.tensor([slot, 0], dtype=torch.int32, device="cuda")
    ins = [synth.host_to_torch(x, BF16) for x in (q, kn, vn)]
    if paged:
        per = (n + page - 1) // page
        pool = lambda X: torch.cat([X, X.new_zeros(P, Hkv, per * page - n, d)], 2).reshape(P, Hkv, per, page, d).transpose(1, 2).reshape(
            P * per, Hkv, page, d).contiguous()
        Kp, Vp = pool(Kd), pool(Vd)
        table = torch.arange(P * per, dtype=torch.int32, device="cuda").reshape(P, per)
        sk.sagekv_decode_step_paged(desc, sk.compact_pages(table, Kp, Vp), *ins, Kp, Vp, 0, state, out, ws)
    else:
        sk.sagekv_decode_step_ring(desc, *ins, Kd, Vd, state, out, ws)
    assert state.tolist() == [slot + 1, 0]
    assert np.abs(out.cpu().numpy() - want).max() <= gu.DECODE_ATOL[BF16]


@pytest.mark.parametrize("G", [1, 2, 3, 4, 8])
def test_whole_short_fp32_rows_keep_their_precision(ref, G):
    """A row of 256 tokens in one workgroup of 8 or 16 waves has as many parts to merge.  Each part is good to about 0.8e-7 (2-norm
    over the outputs), which is what two slices of four waves each came to 1.1e-7 with; merged in fp32, 16 waves are at
    1.25e-7 and 8 at 1.13e-7."""
    import torch

    import paper_2503_08879_amd as sk

    P, Hkv, d, n = 8, 2, 64, 256
    rng = np.random.default_rng(G)
    num = den = 0.0
    for _ in range(4):
        q, K, V = (rng.standard_normal(s, dtype=np.float32) for s in ((P, G * Hkv, d), (P, Hkv, n, d), (P, Hkv, n, d)))
        desc, ws, out = gu.gpu_decode_setup(F32, P, G * Hkv, Hkv, d, 0, 0, n, n)
        sk.sagekv_decode_attn(desc, *(torch.from_numpy(x).cuda() for x in (q, K, V)), n, out, ws)
        l = np.matmul(q.reshape(P, Hkv, G, d).astype(np.float64), K.astype(np.float64).transpose(0, 1, 3, 2)) / 8.0
        w = np.exp(l - l.max(-1, keepdims=True))
        want = np.matmul(w / w.sum(-1, keepdims=True), V.astype(np.float64)).reshape(P, G * Hkv, d)
        num += float(((out.cpu().numpy() - want) ** 2).sum())
        den += float((want ** 2).sum())
    assert (num / den) ** 0.5 <= 1.0e-7
