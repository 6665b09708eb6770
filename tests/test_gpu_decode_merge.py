"""Rows cut into slices and merged again: one slice, a few, the 32 that a round of the merge takes, more; per-query rows, where a
head attends nothing in most slices; the new token of a step, wherever its slot lies in a slice."""
import numpy as np
import pytest

import synth
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu
BF16, F32 = synth.BF16, synth.F32


@pytest.mark.parametrize("dtype,Hq,Hkv,d", [(BF16, 8, 2, 128), (BF16, 7, 1, 64), (BF16, 12, 1, 128), (F32, 4, 2, 64), (F32, 4, 1, 128)])
@pytest.mark.parametrize("slices", [2, 3, 31, 32, 33, 65])
@pytest.mark.parametrize("per_query", [False, True])
def test_slices(ref, dtype, Hq, Hkv, d, slices, per_query):
    import paper_2503_08879_amd as sk

    P, G = 1, Hq // Hkv
    n = 128 * slices - 45  # the last slice is ragged
    S, lists = 3, G if per_query else 1
    k = (n - S - 20) // lists
    W = n - S - lists * k
    rng = np.random.default_rng(slices * 100 + Hq + d)
    draw = lambda *shape: synth.round_to_dtype(rng.standard_normal(shape, dtype=np.float32), dtype)
    q, Kc, Vc = draw(P, Hq, d), draw(P, Hkv, n, d), draw(P, Hkv, n, d)
    desc, ws, out = gu.gpu_decode_setup(dtype, P, Hq, Hkv, d, S, k, W, n, head_mode=int(per_query))
    want = ref.decode_attn(dtype, int(per_query), q, Kc, Vc, n, S, k, W)
    sk.sagekv_decode_attn(desc, *(synth.host_to_torch(x, dtype) for x in (q, Kc, Vc)), n, out, ws)
    gu.check_decode(out.cpu().numpy(), want, dtype)


@pytest.mark.parametrize("dtype,Hq,Hkv,d", [(BF16, 8, 2, 128), (BF16, 7, 1, 64), (F32, 4, 2, 64), (F32, 4, 1, 128)])
@pytest.mark.parametrize("slices", [7, 8, 16, 24, 31, 32, 40])
@pytest.mark.parametrize("slice_of", [0, -1])
def test_infinite_value(ref, dtype, Hq, Hkv, d, slices, slice_of):
    """A value of +inf in the first or the last slice is that dim's output, not NaN: a slice enters the sum once."""
    import paper_2503_08879_amd as sk

    P, G, n, S = 1, Hq // Hkv, 128 * slices - 45, 3
    W = 20
    k = n - S - W
    rng = np.random.default_rng(slices + Hq + d)
    draw = lambda *shape: synth.round_to_dtype(rng.standard_normal(shape, dtype=np.float32), dtype)
    q, Kc, Vc = draw(P, Hq, d), draw(P, Hkv, n, d), draw(P, Hkv, n, d)
    Vc[0, 0, 10 if slice_of == 0 else n - 30, 5] = 0x7F80 if dtype == BF16 else np.inf
    desc, ws, out = gu.gpu_decode_setup(dtype, P, Hq, Hkv, d, S, k, W, n)
    sk.sagekv_decode_attn(desc, *(synth.host_to_torch(x, dtype) for x in (q, Kc, Vc)), n, out, ws)
    got = out.cpu().numpy()
    assert np.isposinf(got[0, :G, 5]).all()
    want = ref.decode_attn(dtype, 0, q, Kc, Vc, n, S, k, W)
    np.testing.assert_array_equal(np.isinf(got), np.isinf(want))
    fin = np.isfinite(want)
    assert np.abs(got[fin] - want[fin]).max() <= gu.DECODE_ATOL[dtype]


@pytest.mark.parametrize("dtype,Hq,d", [(BF16, 2, 128), (BF16, 3, 64), (BF16, 7, 128), (F32, 2, 64), (F32, 3, 128)])
@pytest.mark.parametrize("slices", [17, 24, 33, 65])
@pytest.mark.parametrize("S", [0, 3])
@pytest.mark.parametrize("bad", [np.inf, np.nan])
def test_value_of_another_heads_list(ref, dtype, Hq, d, slices, S, bad):
    """Per-query rows: what is no number in slices where a head attends nothing does not reach that head."""
    import paper_2503_08879_amd as sk

    n, W = 128 * slices - 45, 20
    k = (n - S - W) // Hq
    W = n - S - Hq * k
    rng = np.random.default_rng(slices + Hq + d)
    draw = lambda *shape: synth.round_to_dtype(rng.standard_normal(shape, dtype=np.float32), dtype)
    q, Kc, Vc = draw(1, Hq, d), draw(1, 1, n, d), draw(1, 1, n, d)
    assert S + k >= 256  # the second slice is head 0's alone
    Vc[0, 0, 200, 5] = synth.round_to_dtype(np.array([bad], np.float32), dtype)[0]
    desc, ws, out = gu.gpu_decode_setup(dtype, 1, Hq, 1, d, S, k, W, n, head_mode=1)
    sk.sagekv_decode_attn(desc, *(synth.host_to_torch(x, dtype) for x in (q, Kc, Vc)), n, out, ws)
    got, want = out.cpu().numpy(), ref.decode_attn(dtype, 1, q, Kc, Vc, n, S, k, W)
    assert np.isfinite(got[0, 1:]).all() and not np.isfinite(got[0, 0, 5])
    gu.check_decode(got[0, 1:], want[0, 1:], dtype)


FEW = [(BF16, 1, 8, 2, 128), (BF16, 2, 7, 1, 64), (BF16, 1, 12, 1, 128), (F32, 1, 4, 2, 64)]
MANY = [(BF16, 192, 7, 1, 128), (BF16, 192, 12, 1, 64), (BF16, 257, 5, 1, 64)]  # whole rows, in 8 waves and in 4


@pytest.mark.parametrize("dtype,P,Hq,Hkv,d,slices", [(*f, s) for f in FEW for s in (3, 33)] + [(*m, 3) for m in MANY])
@pytest.mark.parametrize("at", ["row start", "slice start", "mid row", "last slice", "row end"])
@pytest.mark.parametrize("call", ["step", "ring", "paged", "paged ring"])
def test_new_token(ref, dtype, P, Hq, Hkv, d, slices, at, call):
    """The new token holds about a third of every head's mass: without it in the keys or in the values the output would be off by about
    its own size (the slices of few rows have 128 tokens, the last one is ragged)."""
    import torch

    import paper_2503_08879_amd as sk

    n, G = 128 * slices - 45, Hq // Hkv
    slot = {"row start": 0, "slice start": 128, "mid row": 205, "last slice": 128 * (slices - 1), "row end": n - 1}[at]
    rng = np.random.default_rng(slices * 100 + Hq + d + slot)
    draw = lambda *shape: synth.round_to_dtype(rng.standard_normal(shape, dtype=np.float32), dtype)
    q, Kc, Vc, vn = draw(P, Hq, d), draw(P, Hkv, n, d), draw(P, Hkv, n, d), draw(P, Hkv, d)
    # the key of least norm whose logit with each query of its group is log(n) (the others' exponentials add up to 1.6 n on average)
    qf = synth.to_f64(q, dtype).reshape(P, Hkv, G, d)
    kn = synth.round_to_dtype((np.linalg.pinv(qf) @ np.full((P, Hkv, G, 1), np.log(0.8 * n) * d ** 0.5))[..., 0], dtype)
    Kd, Vd = synth.host_to_torch(Kc, dtype), synth.host_to_torch(Vc, dtype)
    Kc[:, :, slot], Vc[:, :, slot] = kn, vn
    want = ref.decode_attn(dtype, 0, q, Kc, Vc, n)
    desc, ws, out = gu.gpu_decode_setup(dtype, P, Hq, Hkv, d, 0, 0, n, n)  # the whole row is the window
    ins = [synth.host_to_torch(x, dtype) for x in (q, kn, vn)]
    state = torch.tensor([slot, 0], dtype=torch.int32, device="cuda") if "ring" in call else None
    if "paged" in call:
        per = -(-n // 16)
        table = torch.randperm(P * per).to(torch.int32).reshape(P, per).cuda()

        def pool(X):
            out = torch.full((P * per, Hkv, 16, d), float("nan"), dtype=X.dtype, device="cuda")
            X = torch.cat([X, X.new_full((P, Hkv, per * 16 - n, d), float("nan"))], 2)
            out[table.long().reshape(-1)] = X.reshape(P, Hkv, per, 16, d).transpose(1, 2).reshape(P * per, Hkv, 16, d)
            return out

        Kp, Vp = pool(Kd), pool(Vd)
        sk.sagekv_decode_step_paged(desc, sk.compact_pages(table, Kp, Vp), *ins, Kp, Vp, slot, state, out, ws)
    elif state is not None:
        sk.sagekv_decode_step_ring(desc, *ins, Kd, Vd, state, out, ws)
    else:
        sk.sagekv_decode_step(desc, *ins, Kd, Vd, slot, out, ws)
    gu.check_decode(out.cpu().numpy(), want, dtype)
