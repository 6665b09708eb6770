"""Logits that share an offset, as keys with a common component have them: thousands of a row's softmax terms are heavy, each of them a little.
Rows that one workgroup selects from list them again with a higher threshold (raise_thresholds), longer ones have them taken by workgroups of their own;
sizes on both sides of the lists, rows whose terms no threshold can thin out, and what such calls may cost beside logits around 0."""
import numpy as np
import pytest

import synth
from tests import test_gpu_parity as parity
from tests.test_gpu_row_select import offset_case
from tests.test_gpu_shortlist import check

pytestmark = pytest.mark.gpu
BF16, F32 = synth.BF16, synth.F32
DENSE = 1


@pytest.mark.parametrize("dtype,P,Hq,Hkv,d,L,head_mode", [
    (BF16, 2, 4, 4, 128, 8191, 0),    # one head: 1700 terms, 200 with the higher threshold
    (BF16, 1, 8, 2, 128, 8192, 0),    # 6600, 820
    (BF16, 1, 16, 1, 64, 4097, 0),    # 24000, 4500: about what the list takes
    (BF16, 1, 40, 1, 64, 2050, 0),    # 40 heads: more than it takes
    (BF16, 1, 7, 1, 128, 8000, 1),    # a list per head
    (BF16, 2, 8, 2, 64, 2000, 0),
    (BF16, 1, 4, 1, 64, 24570, 0),
    (F32, 1, 8, 2, 128, 6001, 0),
    (F32, 1, 9, 1, 64, 3000, 1),
    (BF16, 1, 8, 2, 128, 8193, 0),    # rows spread over several workgroups: one more workgroup per head
    (BF16, 1, 40, 2, 64, 24577, 0),   # one per head, 20 of them
    (BF16, 7, 28, 4, 64, 30001, 0),   # one for several heads
    (BF16, 1, 7, 1, 128, 20000, 1),
    (F32, 1, 6, 2, 128, 26000, 0),
])
@pytest.mark.parametrize("offset,scale", [(60.0, 1.0), (-200.0, 1.0), (40.0, 3.0)])
def test_offset_rows(ref, dtype, P, Hq, Hkv, d, L, head_mode, offset, scale):
    q, K, V = offset_case(L, P, Hq, Hkv, d, L, dtype, offset, scale)
    outs = [check(ref, dtype, head_mode, q, K, V, 4, 64, L // 11, flags=DENSE) for _ in range(2)]
    np.testing.assert_array_equal(outs[0]["kept"], outs[1]["kept"])


@pytest.mark.parametrize("dtype,Hq,n_heavy", [(BF16, 8, 65), (BF16, 8, 511), (BF16, 8, 513), (BF16, 2, 2048), (BF16, 2, 2049), (F32, 8, 600)])
def test_terms_that_no_threshold_thins_out(ref, dtype, Hq, n_heavy):
    """n_heavy tokens with the same logit near 36 for each of Hq heads: all of them above any threshold, 520 to 4800 terms for the list's 4096 places."""
    L, S, W, k, d = 7000, 4, 64, 900, 64
    q, K, V = parity.rand_case(n_heavy, 1, Hq, 1, d, L, dtype)
    Kf, qf = synth.to_f64(K, dtype), synth.to_f64(q, dtype)
    at = np.random.default_rng(n_heavy).permutation(L)[:n_heavy]
    Kf[0, 0, at] = np.linalg.pinv(qf[0]) @ np.full(Hq, 36.0 * d ** 0.5) + 0.01 * Kf[0, 0, at]
    check(ref, dtype, 0, q, synth.round_to_dtype(Kf, dtype), V, S, W, k, flags=DENSE)


def whole_pass(P, Hq, Hkv, d, L, k, offset):
    """Best time of a pass over logits of N(offset, 1), us."""
    import torch

    import paper_2503_08879_amd as sk

    S, W = 4, 64
    g = torch.Generator(device="cuda")
    g.manual_seed(L)
    q = torch.randn((P, Hq, d), generator=g, device="cuda").bfloat16()
    K, V = (torch.randn((P, Hkv, L, d), generator=g, device="cuda", dtype=torch.bfloat16) for _ in range(2))
    heads = q.double().reshape(P, Hkv, Hq // Hkv, d).cpu()
    u = torch.linalg.pinv(heads) @ torch.full((P, Hkv, Hq // Hkv, 1), offset * d ** 0.5, dtype=torch.float64)
    K += u[..., 0].unsqueeze(2).to(K)
    desc = sk.select_desc(q, K, V, S, W, k)
    ws = torch.empty(sk.sagekv_select_workspace_bytes(desc), dtype=torch.uint8, device="cuda")
    Kc = torch.empty((P, Hkv, S + k + W, d), dtype=K.dtype, device="cuda")
    Vc = torch.empty_like(Kc)
    kept = torch.empty((P, Hkv, S + k + W), dtype=torch.int32, device="cuda")
    best = 1e9
    for _ in range(8):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(10):
            sk.sagekv_select(desc, q, K, V, Kc, Vc, kept, None, ws)
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b) * 100)
    return best


@pytest.mark.parametrize("P,Hq,Hkv,d,L,k,most", [
    (1, 32, 8, 128, 8192, 700, 3.0),   # N(0, 1) and N(60, 1): 24.4 and 50.5 us, 2.1 times (with every heavy term taken, 5.8 times)
    (8, 128, 8, 128, 8192, 700, 3.3),  # 77 and 181, 2.4 (6.9)
    (8, 32, 8, 128, 2048, 188, 3.2),   # 24.9 and 56.6, 2.3 (5.9)
    (1, 32, 8, 128, 32768, 1788, 1.6),   # 39.3 and 44.7, 1.14 (one workgroup per list for every term: 2.4)
    (1, 128, 8, 128, 32768, 1788, 1.5),  # 53 and 55, 1.03 (5.0)
    (8, 28, 4, 128, 32768, 1788, 1.5),   # 92 and 103, 1.12 (2.0)
])
def test_an_offset_costs_little(P, Hq, Hkv, d, L, k, most):
    times = [whole_pass(P, Hq, Hkv, d, L, k, offset) for offset in (0.0, 60.0)]
    assert times[1] < most * times[0], times
