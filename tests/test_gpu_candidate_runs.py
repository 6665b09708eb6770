"""The filtering pass stores a wave's candidates in runs: none, one run, many (whole blocks of 64 tokens pass), and clusters
that use a chunk's own slots up and go on in the row's pool.  Groups padded to 4, 8 and 16 heads; chunks of 256 to 1024 tokens.
(As they are, these calls take the one-sweep path; test_gpu_filter_route has them on the pre-filtered one.)"""
import numpy as np
import pytest

import synth
from tests import gpu_util as gu
from tests.test_gpu_parity import rand_case

pytestmark = pytest.mark.gpu
BF16 = synth.BF16


@pytest.mark.parametrize("Hq,Hkv,d,P,L", [
    (4, 1, 64, 1, 20001),    # chunks of 256 tokens
    (16, 8, 64, 1, 40000),   # 512
    (32, 8, 64, 2, 40003),   # 1024
    (7, 1, 128, 1, 33000),
    (56, 8, 64, 2, 33001),
    (12, 1, 128, 1, 33000),
    (32, 2, 64, 2, 70001),
])
@pytest.mark.parametrize("head_mode", [0, 1])
def test_crowded_candidates(ref, Hq, Hkv, d, P, L, head_mode):
    S, W, G = 4, 64, Hq // Hkv
    lists = G if head_mode else 1
    k = 1500 // lists
    q, K, V = rand_case(Hq * 10 + d + P, P, Hq, Hkv, d, L, BF16)
    qf, Kf = synth.to_f64(q, BF16).reshape(P, Hkv, G, d), synth.to_f64(K, BF16).reshape(P, Hkv, L, d)
    u = qf.mean(2) / np.linalg.norm(qf.mean(2), axis=-1, keepdims=True)
    # one crowd per row: 40 tokens, a whole block and its neighbours, or 1100 in one piece, across the edges of chunks
    for p in range(P):
        for c in range(Hkv):
            n = (40, 300, 1100)[(p * Hkv + c) % 3]
            at = 3 * 1024 - 20 + 64 * c
            Kf[p, c, at:at + n] += 1.5 * u[p, c]
    K = synth.round_to_dtype(Kf.reshape(K.shape), BF16)
    Kc, _, kept, s = ref.select(BF16, head_mode, q, K, V, S, W, k, want_scores=True)
    out = gu.gpu_select(BF16, q, K, V, S, W, k, want_scores=False, head_mode=head_mode)
    assert out["redone"] == 0  # nothing was lost on the way: no row needed the dense path
    exempt = 0
    for li in range(lists):
        cut = lambda a: np.concatenate([a[..., :S], a[..., S + li * k:S + (li + 1) * k], a[..., S + lists * k:]], axis=-1)
        exempt += gu.check_kept(cut(out["kept"]), cut(kept), s.reshape(P, Hkv, lists, L)[:, :, li], S, W, k)
    if exempt == 0:
        np.testing.assert_array_equal(out["Kc"], Kc)
