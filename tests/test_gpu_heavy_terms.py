"""Softmax terms that the filtering and partials passes take with an fp64 exponent: planted at the edges of tiles, blocks and
chunks, in the ragged last block, one head at a time.  A term that is missed, taken twice or given to another head would put that
head's scores off by the term's share of the mass (several per cent).  The partials pass's scores are held to 1e-5.  What the filtering pass
made of them shows in its kept sets, summed over heads of unlike normalisers, and in that no row had to be redone.  (As they are, the calls without scores
take the one-sweep path; test_gpu_filter_route has them on the pre-filtered one.)"""
import numpy as np
import pytest

import synth
from tests import gpu_util as gu
from tests.test_gpu_parity import rand_case

pytestmark = pytest.mark.gpu
BF16 = synth.BF16


@pytest.mark.parametrize("G,d", [(1, 64), (3, 128), (4, 128), (5, 64), (7, 128), (8, 64), (12, 128), (16, 64), (16, 128)])
@pytest.mark.parametrize("L", [4099, 30017])
def test_planted_heavy_terms(ref, G, d, L):
    S, W, k, Hkv = 4, 64, 100 if G <= 8 else 20, 3  # (a k the pre-filter takes for every list)
    q, K, V = rand_case(G * 100 + d + L, 1, G * Hkv, Hkv, d, L, BF16)
    qf, Kf = synth.to_f64(q, BF16).reshape(Hkv, G, d), synth.to_f64(K, BF16).reshape(Hkv, L, d)
    at = [0, 15, 16, 63, 64, 255, 256, 1023, 1024, 1041, L // 2, L - W - 1, L - 17, L - 2, L - 1]
    for c in range(Hkv):
        for i, t in enumerate(at):
            g = (i + c) % G
            u = qf[c, g] / np.linalg.norm(qf[c, g])
            Kf[c, t] = (7.0 + 0.1 * i) * u + 0.1 * Kf[c, t]  # a logit of 7 to 8.5: 4 to 15 per cent of a head's mass each at L = 4099
    K = synth.round_to_dtype(Kf.reshape(K.shape), BF16)
    Kc, _, kept, s = ref.select(BF16, 1, q, K, V, S, W, k, want_scores=True)
    out = gu.gpu_select(BF16, q, K, V, S, W, k, want_scores=True, head_mode=1)  # every head's own probabilities
    gu.check_scores(out["scores"], s.reshape(out["scores"].shape))
    for head_mode in (0, 1):
        lists = G if head_mode else 1
        Kc, _, kept, s = ref.select(BF16, head_mode, q, K, V, S, W, k, want_scores=True)
        out = gu.gpu_select(BF16, q, K, V, S, W, k, want_scores=False, head_mode=head_mode)
        assert out["redone"] == 0  # the path's own result: no row went another way
        for li in range(lists):
            cut = lambda a: np.concatenate([a[..., :S], a[..., S + li * k:S + (li + 1) * k], a[..., S + lists * k:]], axis=-1)
            gu.check_kept(cut(out["kept"]), cut(kept), s.reshape(1, Hkv, lists, L)[:, :, li], S, W, k)


@pytest.mark.parametrize("G,d", [(1, 128), (3, 64), (4, 128), (7, 64), (8, 128), (12, 64), (16, 128)])
@pytest.mark.parametrize("L", [4099, 30017])
def test_terms_strewn_thin(ref, G, d, L):
    """Logits that share an offset: where |M| is 60, one token in a hundred is heavy, so that tiles hold none, one or a few terms;
    beside them tiles that are full of terms, one head's or all heads'."""
    S, W, k, Hkv = 4, 64, 100 if G <= 8 else 20, 3
    q, K, V = rand_case(G * 100 + d + L + 1, 1, G * Hkv, Hkv, d, L, BF16)
    qf, Kf = synth.to_f64(q, BF16).reshape(Hkv, G, d), synth.to_f64(K, BF16).reshape(Hkv, L, d)
    for c in range(Hkv):
        Kf[c] += np.linalg.pinv(qf[c]) @ np.full(G, (60.0, -45.0, 30.0)[c] * d ** 0.5)  # every head's logits around that
        for g in range(G):
            Kf[c, 640 + 16 * (g % 4):656 + 16 * (g % 4)] += 2.5 * qf[c, g] / np.linalg.norm(qf[c, g])
    K = synth.round_to_dtype(Kf.reshape(K.shape), BF16)
    for head_mode in (0, 1):
        lists = G if head_mode else 1
        Kc, _, kept, s = ref.select(BF16, head_mode, q, K, V, S, W, k, want_scores=True)
        for want_scores in (True, False):
            out = gu.gpu_select(BF16, q, K, V, S, W, k, want_scores=want_scores, head_mode=head_mode)
            if want_scores:
                # an fp32 logit of 60 to 64, a sum of 128 products in units of up to 2^-18, is off by up to 1.5e-5, and a score by as much of
                # itself; what all of a head's scores have in common, its normaliser's error among it, differs between heads by less
                # than the scores that may change places (a heavy term has 1e-4 of a head's mass or more)
                rel = out["scores"].reshape(s.shape).astype(np.float64) / s - 1.0
                assert np.abs(rel).max() <= 3e-5
                assert np.ptp(rel.mean(-1), axis=-1).max() <= gu.TIE_RTOL
            else:
                assert out["redone"] == 0
            for li in range(lists):
                cut = lambda a: np.concatenate([a[..., :S], a[..., S + li * k:S + (li + 1) * k], a[..., S + lists * k:]], axis=-1)
                gu.check_kept(cut(out["kept"]), cut(kept), s.reshape(1, Hkv, lists, L)[:, :, li], S, W, k)


@pytest.mark.parametrize("Hq,Hkv,d,at_most", [(32, 8, 128, 1.25), (28, 4, 64, 1.5)])
def test_an_offset_costs_little(Hq, Hkv, d, at_most):
    """The pass over logits N(60, 1) against N(0, 1): 1.0 (4 heads of 128 dims) and 1.2 to 1.3 (7 of 64) times as long with the terms
    taken one by one, 1.5 and 1.8 with whole tiles' products for each of them."""
    import torch

    import paper_2503_08879_amd as sk

    P, L, S, W, k, G = 256 // Hkv, 32768, 4, 256, 1788, Hq // Hkv
    g = torch.Generator(device="cuda")
    g.manual_seed(Hq)
    q = torch.randn((P, Hq, d), generator=g, device="cuda").bfloat16()
    K, V = (torch.randn((P, Hkv, L, d), generator=g, device="cuda", dtype=torch.bfloat16) for _ in range(2))
    shift = torch.linalg.pinv(q.float().reshape(P, Hkv, G, d)) @ torch.full((P, Hkv, G, 1), 60.0 * d ** 0.5, device="cuda")
    desc = sk.select_desc(q, K, V, S, W, k, S + k + W)
    ws = torch.empty(sk.sagekv_select_workspace_bytes(desc), dtype=torch.uint8, device="cuda")
    Kc = torch.zeros((P, Hkv, S + k + W, d), dtype=torch.bfloat16, device="cuda")
    Vc, kept = torch.zeros_like(Kc), torch.zeros((P, Hkv, S + k + W), dtype=torch.int32, device="cuda")
    times = []
    for _ in range(2):
        laps = []
        for _ in range(15):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(3):
                sk.sagekv_select(desc, q, K, V, Kc, Vc, kept, None, ws)
            b.record()
            torch.cuda.synchronize()
            laps.append(a.elapsed_time(b))
        assert sk.sagekv_select_redone_rows(desc, ws) == 0
        times.append(sorted(laps)[len(laps) // 2])
        K += shift.reshape(P, Hkv, 1, d).bfloat16()
    assert times[1] <= at_most * times[0], times
