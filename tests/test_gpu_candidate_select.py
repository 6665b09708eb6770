"""The pre-filtered path's candidate selection: rows whose candidates fit the registers of the workgroup that owns them (4,
12 or 24 per thread, by what a list is expected to have), and peaked rows that have more and go through memory.  As they are, most of these calls are
small enough for the one-sweep path; test_gpu_filter_route has them on the pre-filtered one."""
import numpy as np
import pytest

import synth
from tests import gpu_util as gu
from tests.test_gpu_parity import rand_case

pytestmark = pytest.mark.gpu
BF16 = synth.BF16


@pytest.mark.parametrize("scale", [1.0, 4.0])  # 4: heavy-tailed rows take up to twice the planned candidates
@pytest.mark.parametrize("Hq,Hkv,d,L,ks,head_mode", [
    (8, 2, 128, 65536, (1, 900, 1500, 1900, 4500, 6000), 0),   # 4 heads: 2 to 14 thousand candidates
    (16, 2, 64, 65537, (1000, 1800, 5000), 0),                 # 8 heads
    (12, 1, 128, 50001, (700, 1500, 3000), 0),                 # 12 heads: records padded to 16
    (16, 1, 64, 120001, (1000, 3000), 0),                      # 16 heads, a sample of more than 9 items per thread
    (4, 1, 64, 200000, (9000,), 0),                            # more than 12288 expected
    (7, 1, 128, 65536, (1, 300, 1500), 1),                     # per-query lists
])
def test_candidate_counts_around_the_register_sizes(ref, Hq, Hkv, d, L, ks, head_mode, scale):
    S, W = 4, 64
    G = Hq // Hkv
    lists = G if head_mode else 1
    q, K, V = rand_case(Hq * 1000 + d, 1, Hq, Hkv, d, L, BF16)
    q = synth.round_to_dtype(scale * synth.to_f64(q, BF16), BF16)
    for k in ks:
        Kc, _, kept, s = ref.select(BF16, head_mode, q, K, V, S, W, k, want_scores=True)
        out = gu.gpu_select(BF16, q, K, V, S, W, k, want_scores=False, head_mode=head_mode)
        assert out["redone"] >= 0  # not a dense call
        if scale == 1.0:
            assert out["redone"] == 0
        exempt = 0
        for li in range(lists):
            cut = lambda a: np.concatenate([a[..., :S], a[..., S + li * k:S + (li + 1) * k], a[..., S + lists * k:]], axis=-1)
            exempt += gu.check_kept(cut(out["kept"]), cut(kept), s[:, :, li], S, W, k)
        if exempt == 0:
            np.testing.assert_array_equal(out["Kc"], Kc)
