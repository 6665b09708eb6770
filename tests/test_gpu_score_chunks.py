"""Calls large enough for the score pass's larger chunks: 1024 tokens per workgroup (bf16) and 512 (fp32), which take 512
workgroups (256 in a dense call that returns the scores); with rows of several chunks and ragged ends.  (test_gpu_filter_route has the filtered
ones on the pre-filtered path whatever their size.)"""
import pytest

import synth
from tests import gpu_util as gu
from tests.test_gpu_paged import paged_case
from tests.test_gpu_parity import rand_case
from tests.test_gpu_row_select import parity

pytestmark = pytest.mark.gpu
BF16, F32 = synth.BF16, synth.F32


@pytest.mark.parametrize("dtype,chunk,G,d,L,head_mode", [
    (BF16, 1024, 4, 128, 8192, 0), (BF16, 1024, 7, 64, 4097, 0), (BF16, 1024, 12, 128, 8191, 0),
    (BF16, 1024, 4, 64, 4097, 1), (BF16, 1024, 7, 128, 8192, 1), (BF16, 1024, 12, 64, 8191, 1),
    (BF16, 1024, 20, 64, 4097, 0),
    (F32, 512, 4, 64, 8191, 0), (F32, 512, 8, 128, 4097, 0), (F32, 512, 3, 64, 4097, 1),
])
def test_dense_rows_of_full_chunks(ref, dtype, chunk, G, d, L, head_mode):
    P, Hkv = 32, 2
    assert P * Hkv * -(-L // chunk) >= 256
    q, K, V = rand_case(L + G, P, G * Hkv, Hkv, d, L, dtype)
    parity(ref, dtype, head_mode, q, K, V, 4, 100, L // 8)


def test_long_dense_rows_of_full_chunks(ref):
    P, Hq, Hkv, d, L = 4, 8, 2, 64, 33001  # statistics, scores and selection in launches of their own
    assert P * Hkv * -(-L // 1024) >= 256
    q, K, V = rand_case(5, P, Hq, Hkv, d, L, BF16)
    parity(ref, BF16, 0, q, K, V, 4, 100, 3000)


@pytest.mark.parametrize("G,d,page", [(7, 128, 16), (4, 64, 64), (12, 64, 16), (16, 128, 32)])
@pytest.mark.parametrize("want_scores", [False, True])  # the filtering pass; partials, then scores
def test_paged_rows_of_full_chunks(ref, G, d, page, want_scores):
    P, Hkv, L = 8, 2, 32777
    assert P * Hkv * -(-L // 1024) >= 512
    paged_case(ref, BF16, P, G * Hkv, Hkv, d, L, 4, 100, 700, page, token_major=False, want_scores=want_scores, seed=G + d)


@pytest.mark.parametrize("G,d", [(4, 128), (8, 64), (12, 128), (16, 64)])
def test_filtered_rows_of_full_chunks(ref, G, d):
    P, Hkv, L, S, W, k = 8, 2, 32777, 4, 100, 700
    q, K, V = rand_case(G + d, P, G * Hkv, Hkv, d, L, BF16)
    _, _, kept, s = ref.select(BF16, 0, q, K, V, S, W, k, want_scores=True)
    out = gu.gpu_select(BF16, q, K, V, S, W, k, want_scores=False)
    assert out["redone"] == 0
    gu.check_kept(out["kept"], kept, s[:, :, 0], S, W, k)
