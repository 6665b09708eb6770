"""The one-sweep dense path: rows whose scores one workgroup holds in registers (up to 24576 tokens, four sizes), the
longer ones behind them, and the softmax terms that a score chunk takes with fp64 exponents."""
import numpy as np
import pytest

import synth
from tests import gpu_util as gu
from tests.test_gpu_parity import rand_case

pytestmark = pytest.mark.gpu
BF16, F32 = synth.BF16, synth.F32
DENSE = 1


def parity(ref, dtype, head_mode, q, K, V, S, W, k, scores=(False, True)):
    """Kept sets of the dense path, with and without the scores written out, against the oracle's."""
    G = q.shape[1] // K.shape[1]
    lists = G if head_mode else 1
    Kc, _, kept, s = ref.select(dtype, head_mode, q, K, V, S, W, k, want_scores=True)
    for want_scores in scores:
        out = gu.gpu_select(dtype, q, K, V, S, W, k, want_scores=want_scores, flags=DENSE, head_mode=head_mode)
        exempt = 0
        for li in range(lists):
            cut = lambda a: np.concatenate([a[..., :S], a[..., S + li * k:S + (li + 1) * k], a[..., S + lists * k:]], axis=-1)
            exempt += gu.check_kept(cut(out["kept"]), cut(kept), s[:, :, li], S, W, k)
        if exempt == 0:
            np.testing.assert_array_equal(out["Kc"][:, :, : S + lists * k + W], Kc)
        if want_scores:
            gu.check_scores(out["scores"].reshape(s.shape), s)


@pytest.mark.parametrize("dtype,Hq,Hkv,d,head_mode", [(BF16, 8, 2, 128, 0), (F32, 4, 2, 64, 0), (BF16, 7, 1, 64, 1), (F32, 20, 1, 128, 0)])
@pytest.mark.parametrize("L", [9, 255, 4096, 4097, 8192, 8193, 16384, 16389, 24576, 24577])
def test_row_lengths_around_the_register_sizes(ref, dtype, Hq, Hkv, d, head_mode, L):
    S, W = min(3, L // 4), max(1, L // 50)
    E = L - S - W
    q, K, V = rand_case(L + Hq, 1, Hq, Hkv, d, L, dtype)
    for k in sorted({1, E // 4 + 1, E - 1}):
        parity(ref, dtype, head_mode, q, K, V, S, W, k)


@pytest.mark.parametrize("L", [700, 9001, 30000])
def test_thousands_of_equal_scores(ref, L):
    """q = 0 (every score equal) and keys that repeat eight rows (every score L / 8 times): more near-ties than the band
    holds; equal scores go to the lowest positions."""
    P, Hq, Hkv, d, S, W = 1, 8, 2, 64, 2, 5
    q, K, V = rand_case(L, P, Hq, Hkv, d, L, BF16)
    K[:] = K[:, :, np.arange(L) % 8]
    for scale in (0.0, 1.0):
        qs = synth.round_to_dtype(scale * synth.to_f64(q, BF16), BF16)
        for k in (1, L // 3, L - S - W - 1):
            parity(ref, BF16, 0, qs, K, V, S, W, k)


@pytest.mark.parametrize("dtype,flags,L", [(BF16, DENSE, 6000), (F32, 0, 6000), (BF16, 0, 40000), (BF16, DENSE, 40000)])
def test_many_heavy_terms_in_one_chunk(ref, dtype, flags, L):
    """Peaked attention (queries x 6) and 120 heavy tokens side by side: more exact softmax terms than one batch of
    them holds.  The kept set needs every head's normaliser to about 1e-7."""
    P, Hq, Hkv, d, S, W, k = 1, 8, 2, 128, 4, 64, 700
    G = Hq // Hkv
    q, K, V = rand_case(L + flags, P, Hq, Hkv, d, L, dtype)
    q64 = 6.0 * synth.to_f64(q, dtype)
    unit = q64.reshape(P, Hkv, G, d)
    unit = unit / np.linalg.norm(unit, axis=-1, keepdims=True)
    K64 = synth.to_f64(K, dtype)
    K64[:, :, 2:122] += 4.0 * unit.sum(2)[:, :, None, :]
    q, K = synth.round_to_dtype(q64, dtype), synth.round_to_dtype(K64, dtype)
    _, _, kept, s = ref.select(dtype, 0, q, K, V, S, W, k, want_scores=True)
    top = np.sort(s[0, :, 0].astype(np.float64), axis=-1)[:, ::-1]
    assert (top[:, :32].sum(1) > 0.3 * G).all()  # a few tokens hold much of the mass
    out = gu.gpu_select(dtype, q, K, V, S, W, k, want_scores=False, flags=flags)
    assert gu.check_kept(out["kept"], kept, s[:, :, 0], S, W, k) == 0


@pytest.mark.parametrize("n_heavy", [1, 40, 250])
def test_rows_with_heavy_terms_are_deterministic(n_heavy):
    """The heavy terms are listed in whatever order the waves meet them; nothing may depend on it."""
    P, Hq, Hkv, d, L, S, W, k = 4, 8, 4, 64, 8000, 4, 64, 900
    q, K, V = rand_case(n_heavy, P, Hq, Hkv, d, L, BF16)
    G = Hq // Hkv
    Q = synth.to_f64(q, BF16).reshape(P, Hkv, G, d)
    Kf = synth.to_f64(K, BF16)
    u = (np.linalg.pinv(Q) @ np.full((P, Hkv, G, 1), 36.0 * d ** 0.5))[..., 0]
    at = np.random.default_rng(n_heavy).permutation(L)[:n_heavy]
    Kf[:, :, at] = u[:, :, None] + 0.01 * Kf[:, :, at]  # both heads' logits near 36
    K = synth.round_to_dtype(Kf, BF16)
    first = gu.gpu_select(BF16, q, K, V, S, W, k, want_scores=False, flags=DENSE)
    for _ in range(6):
        again = gu.gpu_select(BF16, q, K, V, S, W, k, want_scores=False, flags=DENSE)
        for name in ("kept", "Kc", "Vc"):
            np.testing.assert_array_equal(first[name], again[name])


def offset_case(seed, P, Hq, Hkv, d, L, dtype, offset, scale=1.0):
    """q, K, V with logits of about N(offset, scale): every key has a common component, as trained models' keys do."""
    q, K, V = rand_case(seed, P, Hq, Hkv, d, L, dtype)
    G = Hq // Hkv
    q64 = scale * synth.to_f64(q, dtype)
    Q = q64.reshape(P, Hkv, G, d)
    gram = Q @ Q.transpose(0, 1, 3, 2)
    u = np.linalg.solve(gram, np.full((P, Hkv, G, 1), offset * np.sqrt(d))).transpose(0, 1, 3, 2) @ Q  # q . u / sqrt(d) = offset
    return synth.round_to_dtype(q64, dtype), synth.round_to_dtype(synth.to_f64(K, dtype) + u, dtype), V


@pytest.mark.parametrize("dtype,L", [(BF16, 4090), (BF16, 9001), (F32, 6000), (BF16, 30000), (F32, 25001)])
@pytest.mark.parametrize("offset,scale", [(-30.0, 1.0), (25.0, 2.0), (-200.0, 1.0)])
def test_logits_around_an_offset(ref, dtype, L, offset, scale):
    """A head's exact softmax terms are those that are heavy for the row.  At -200 every token is: more than a wave lists at
    a time."""
    q, K, V = offset_case(L, 1, 8, 2, 64, L, dtype, offset, scale)
    # score values: an fp32 logit of magnitude 200 is off by up to 200 x 2.5e-7 = 5e-5, five times what check_scores allows
    parity(ref, dtype, 0, q, K, V, 4, 64, L // 5, scores=(False, True) if abs(offset) < 40 else (False,))


def test_more_heavy_terms_than_are_taken_exactly(ref):
    """Flat logits around -400 over 40000 tokens: the rest keeps its fp32 terms (one list per query head: a head's
    normaliser does not change the order of its own tokens)."""
    S, W, k, L = 4, 64, 500, 40000
    q, K, V = offset_case(11, 1, 4, 1, 64, L, BF16, -400.0)
    Kc, _, kept, s = ref.select(BF16, 1, q, K, V, S, W, k, want_scores=True)
    out = gu.gpu_select(BF16, q, K, V, S, W, k, want_scores=False, flags=DENSE, head_mode=1)
    for li in range(4):
        cut = lambda a: np.concatenate([a[..., :S], a[..., S + li * k:S + (li + 1) * k], a[..., S + 4 * k:]], axis=-1)
        gu.check_kept(cut(out["kept"]), cut(kept), s[:, :, li], S, W, k)


def test_an_offset_costs_a_dense_pass_little():
    """256 rows x 8192 tokens x 4 heads, logits N(-30, 1) against N(0, 1): 0.4 % against 0 % of the terms are heavy for their
    rows, 1.02 times the time.  (Heavy by their share of a chunk, a third of them would be: 3.1 times.)"""
    import torch

    import paper_2503_08879_amd as sk

    P, Hq, Hkv, d, L, S, W, k = 32, 32, 8, 128, 8192, 4, 256, 1788
    times = []
    for offset in (0.0, -30.0):
        q1, K1, V1 = offset_case(3, 1, Hq, Hkv, d, L, BF16, offset)
        q, K, V = (synth.host_to_torch(x, BF16).repeat(P, *[1] * (x.ndim - 1)) for x in (q1, K1, V1))
        desc = sk.select_desc(q, K, V, S, W, k)
        ws = torch.empty(sk.sagekv_select_workspace_bytes(desc), dtype=torch.uint8, device="cuda")
        Kc = torch.empty((P, Hkv, S + k + W, d), dtype=K.dtype, device="cuda")
        Vc = torch.empty_like(Kc)
        kept = torch.empty((P, Hkv, S + k + W), dtype=torch.int32, device="cuda")
        best = 1e9
        for _ in range(8):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(4):
                sk.sagekv_select(desc, q, K, V, Kc, Vc, kept, None, ws)
            b.record()
            torch.cuda.synchronize()
            best = min(best, a.elapsed_time(b) / 4)
        times.append(best)
    assert times[1] < 1.5 * times[0], times
