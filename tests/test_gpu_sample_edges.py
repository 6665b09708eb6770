"""The sample of the pre-filtered path: runs that straddle pages and the row's ends, heads padded to 4, 8 and 16, rows shorter than
the sample itself, a last workgroup with fewer blocks than waves.  A wrong logit there does not change a kept set but sends its row
to the dense path, so the count of redone rows is checked too.  (As they are, most of these calls take the one-sweep path; test_gpu_filter_route has them on the
pre-filtered one.)"""
import pytest

import synth
from tests.test_gpu_paged import paged_case

pytestmark = pytest.mark.gpu
BF16 = synth.BF16


@pytest.mark.parametrize("P,Hq,Hkv,d,L,S,W,k,page", [
    (1, 4, 1, 128, 505, 0, 500, 1, 16),        # a row shorter than its recent blocks
    (1, 8, 2, 64, 700, 4, 600, 4, 16),
    (2, 7, 1, 128, 2049, 1, 65, 100, 16),
    (1, 16, 1, 64, 5003, 64, 512, 100, 32),
    (1, 12, 1, 128, 20011, 4, 129, 500, 64),
    (11, 32, 8, 128, 6001, 4, 512, 200, 16),   # 88 rows x 25 blocks: one in the last workgroup
    (20, 56, 8, 64, 9001, 4, 512, 100, 16),
])
@pytest.mark.parametrize("token_major", [False, True])
def test_sample_edges(ref, P, Hq, Hkv, d, L, S, W, k, page, token_major):
    redone = paged_case(ref, BF16, P, Hq, Hkv, d, L, S, W, k, page, token_major=token_major)
    assert redone == 0
