"""Softmax terms that the filtering and partials passes take with an fp64 exponent: planted at the edges of tiles, blocks and
chunks, in the ragged last block, one head at a time.  A term that is missed, taken twice or given to another head would put that
head's scores off by the term's share of the mass (several per cent).  The partials pass's scores are held to 1e-5.  What the filtering pass
made of them shows in its kept sets, summed over heads of unlike normalisers, and in that no row had to be redone."""
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
        assert out["redone"] == 0  # the filtering pass's own result: no row went to the partials pass
        for li in range(lists):
            cut = lambda a: np.concatenate([a[..., :S], a[..., S + li * k:S + (li + 1) * k], a[..., S + lists * k:]], axis=-1)
            gu.check_kept(cut(out["kept"]), cut(kept), s.reshape(1, Hkv, lists, L)[:, :, li], S, W, k)
