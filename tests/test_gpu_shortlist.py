"""Calls of few rows: the one-sweep path with a row's selection spread over many workgroups.  Sizes at the edges of the parts (4096 and
8192 tokens), of the sample (rows with fewer runs than it takes, no whole run at all) and of the registers; samples that mislead, so that a list
goes through its whole score row; and callers whose workspace only holds what the pre-filtered path needs."""
import ctypes

import numpy as np
import pytest

import synth
from tests import gpu_util as gu
from tests import test_gpu_candidate_runs as runs
from tests import test_gpu_candidate_select as candidates
from tests import test_gpu_heavy_terms as heavy
from tests import test_gpu_parity as parity
from tests import test_gpu_sample_edges as sample
from tests import test_gpu_score_chunks as chunks
from tests.test_gpu_paged import paged_case

pytestmark = pytest.mark.gpu
BF16, F32 = synth.BF16, synth.F32


def check(ref, dtype, head_mode, q, K, V, S, W, k, flags=0, **dev):
    P, Hkv, L = K.shape[:3]
    lists = q.shape[1] // Hkv if head_mode else 1
    Kc, _, kept, s = ref.select(dtype, head_mode, q, K, V, S, W, k, want_scores=True)
    out = gu.gpu_select(dtype, q, K, V, S, W, k, want_scores=False, head_mode=head_mode, flags=flags, **dev)
    exempt = 0
    for li in range(lists):
        cut = lambda a: np.concatenate([a[..., :S], a[..., S + li * k:S + (li + 1) * k], a[..., S + lists * k:]], axis=-1)
        exempt += gu.check_kept(cut(out["kept"]), cut(kept), s.reshape(P, Hkv, lists, L)[:, :, li], S, W, k)
    if exempt == 0:
        np.testing.assert_array_equal(out["Kc"], Kc)
    gu.check_gather(out, K, V, S, k, W)
    return out


@pytest.mark.parametrize("dtype,P,Hq,Hkv,d,L,S,W,k,head_mode", [
    (BF16, 1, 4, 1, 128, 8193, 0, 1, 1, 0),        # one token past the rows of one workgroup and past two parts
    (BF16, 1, 8, 2, 128, 12287, 4, 64, 1000, 0),   # parts of 4096: one token short of three, three, one more
    (BF16, 1, 8, 2, 128, 12288, 3, 61, 1000, 0),
    (BF16, 1, 7, 1, 64, 12289, 17, 15, 1000, 0),
    (BF16, 2, 32, 8, 128, 60001, 4, 64, 500, 0),   # parts of 8192, 4 heads
    (BF16, 4, 28, 4, 64, 65537, 4, 64, 500, 0),    # and 7, ragged
    (BF16, 1, 40, 2, 64, 24577, 4, 64, 300, 0),    # 20 heads: the dense path, eight at a time
    (BF16, 1, 16, 1, 128, 30000, 4, 64, 400, 0),
    (BF16, 1, 7, 1, 128, 9000, 4, 64, 1200, 1),    # a list per head
    (BF16, 1, 28, 4, 64, 40000, 2048, 2560, 512, 1),
    (F32, 1, 4, 2, 64, 9001, 4, 64, 1000, 0),
    (F32, 1, 6, 2, 128, 33333, 4, 64, 300, 1),
    (BF16, 1, 4, 1, 64, 30000, 14980, 15000, 17, 0),   # 20 candidates, no whole run of 16 among them: everything is handed on
    (BF16, 1, 4, 1, 64, 30000, 4, 28000, 1996, 0),     # every candidate selected
    (BF16, 1, 4, 1, 64, 30000, 4, 28000, 1, 0),        # fewer runs than the sample takes
    (BF16, 1, 4, 2, 64, 200000, 4, 64, 9000, 0),       # about 11 thousand handed on: 16 registers
    (F32, 1, 2, 1, 64, 100000, 4, 64, 4000, 0),        # 8
    (BF16, 2, 14, 2, 64, 24600, 4, 64, 4900, 1),       # 28 lists, 224 workgroups: the most but a few for 64 dims
    (BF16, 3, 14, 2, 64, 24600, 4, 64, 4900, 1),       # 42 lists: over that
    (BF16, 4, 28, 4, 128, 24600, 4, 64, 4900, 1),      # 112 lists of 128 dims, 560 workgroups: over that too
    (BF16, 7, 8, 2, 128, 65537, 4, 64, 13200, 0),      # one list per row, 14 lists, 252 workgroups
])
def test_few_rows(ref, dtype, P, Hq, Hkv, d, L, S, W, k, head_mode):
    q, K, V = parity.rand_case(L + Hq + k, P, Hq, Hkv, d, L, dtype)
    out = check(ref, dtype, head_mode, q, K, V, S, W, k)
    assert out["redone"] in (0, -1)  # -1: descriptors that only the dense path serves


@pytest.mark.parametrize("dtype,Hq,L,head_mode", [
    (BF16, 2, 14336, 0), (BF16, 2, 14337, 0), (F32, 4, 12288, 0), (F32, 4, 12289, 0), (BF16, 6, 10240, 0), (BF16, 6, 10241, 0), (F32, 8, 14336, 1), (BF16, 8, 14337, 1)])
def test_around_the_rows_of_one_workgroup(ref, dtype, Hq, L, head_mode):
    """The longest rows that one workgroup selects from and the first ones spread over several, by heads per list."""
    q, K, V = parity.rand_case(L + Hq, 1, Hq, 2, 64, L, dtype)
    check(ref, dtype, head_mode, q, K, V, 4, 64, 700)


@pytest.mark.parametrize("layout", ["token_major", "wide"])
@pytest.mark.parametrize("head_mode", [0, 1])
def test_strided_rows(ref, layout, head_mode):
    import torch

    P, Hq, Hkv, d, L, S, W, k = 2, 8, 2, 128, 12345, 4, 64, 700
    q, K, V = parity.rand_case(3, P, Hq, Hkv, d, L, BF16)
    dev = {}
    for name, X in (("K_dev", K), ("V_dev", V)):
        x = synth.host_to_torch(X, BF16)
        if layout == "token_major":
            x = x.permute(0, 2, 1, 3).contiguous().permute(0, 2, 1, 3)
        else:
            pad = torch.full((P, Hkv, L, d + 24), float("nan"), dtype=x.dtype, device="cuda")
            pad[..., :d] = x
            x = pad[..., :d]
        dev[name] = x
    check(ref, BF16, head_mode, q, K, V, S, W, k, **dev)


@pytest.mark.parametrize("dtype,Hq,Hkv,d,L,page,head_mode", [(BF16, 7, 1, 128, 20011, 16, 0), (BF16, 8, 2, 64, 33000, 64, 1), (F32, 4, 2, 64, 12001, 16, 0)])
def test_paged_rows(ref, dtype, Hq, Hkv, d, L, page, head_mode):
    paged_case(ref, dtype, 2, Hq, Hkv, d, L, 4, 64, 400, page, head_mode=head_mode, token_major=True, seed=L)


@pytest.mark.parametrize("P,Hq,Hkv,L,head_mode", [(1, 8, 2, 8000, 0), (1, 8, 2, 30000, 0), (1, 8, 2, 30000, 1), (2, 4, 2, 100000, 0)])
def test_a_sample_that_misleads(ref, P, Hq, Hkv, L, head_mode):
    """The sampled runs hold the row's largest scores (too few are handed on), its smallest (too many), or all scores tie: the list goes
    through its whole score row.  Rows of ordinary keys beside them do not."""
    S, W, k, d = 0, 16, 600, 64
    q, K, V = parity.rand_case(L, P, Hq, Hkv, d, L, BF16)
    Kf, qf = synth.to_f64(K, BF16), synth.to_f64(q, BF16).reshape(P, Hkv, Hq // Hkv, d)
    step = ((L - W) // 16 << 16) // 128  # the library samples 128 of the candidates' aligned runs
    at = ((np.arange(128) * step >> 16)[:, None] * 16 + np.arange(16)).reshape(-1)
    for kind in ("high", "low", "equal"):
        X = Kf.copy()
        u = qf[0, 0].mean(0) / np.linalg.norm(qf[0, 0].mean(0))
        if kind == "equal":
            X[0, 0] = X[0, 0, :1]
        else:
            X[0, 0, at] += (6.0 if kind == "high" else -12.0) * u
        Kb = synth.round_to_dtype(X, BF16)
        out = check(ref, BF16, head_mode, q, Kb, V, S, W, k)
        assert out["redone"] == (kind == "equal" or L > 8192), kind  # (a shorter row has no sample)


@pytest.mark.parametrize("dtype", [BF16, F32])
@pytest.mark.parametrize("n_heavy", [1, 255, 256, 257, 600])
def test_heavy_terms_around_the_list(ref, dtype, n_heavy):
    """Two heads, n_heavy tokens each with a logit near 36 for both: 2 n_heavy terms for the 512 places where a row's heavy terms are
    listed as its logits pass through the registers."""
    P, Hq, Hkv, d, L, S, W, k = 2, 2, 1, 64, 6001, 4, 64, 900
    q, K, V = parity.rand_case(n_heavy, P, Hq, Hkv, d, L, dtype)
    Kf, qf = synth.to_f64(K, dtype), synth.to_f64(q, dtype)
    at = np.random.default_rng(n_heavy).permutation(L)[:n_heavy]
    for p in range(P):
        u = np.linalg.pinv(qf[p]) @ np.full(Hq, 36.0 * d ** 0.5)
        Kf[p, 0, at] = u + 0.01 * Kf[p, 0, at]
    K = synth.round_to_dtype(Kf, dtype)
    check(ref, dtype, 0, q, K, V, S, W, k, flags=1)


def smallest_workspace(desc):
    """The least that calls with this descriptor accept, found through the call that only reads the workspace's first word."""
    import torch

    import paper_2503_08879_amd as sk

    lib, n = sk.binding.lib(), ctypes.c_int32()
    word = torch.zeros(64, dtype=torch.int32, device="cuda")
    lo, hi = 0, 1 << 40
    while hi - lo > 1:
        mid = (lo + hi) // 2
        code = lib.sagekv_select_redone_rows(ctypes.byref(desc), word.data_ptr(), mid, torch.cuda.current_stream().cuda_stream, ctypes.byref(n))
        assert code in (0, 3)
        lo, hi = (mid, hi) if code == 3 else (lo, mid)
    return hi


@pytest.fixture
def small(monkeypatch):
    import paper_2503_08879_amd as sk

    sizes = []
    full = sk.sagekv_select_workspace_bytes

    def least(desc):
        n = smallest_workspace(desc)
        sizes.append((n, full(desc)))
        return n

    monkeypatch.setattr(sk, "sagekv_select_workspace_bytes", least)
    return sizes


@pytest.mark.parametrize("test,args", [
    (sample.test_sample_edges, (1, 12, 1, 128, 20011, 4, 129, 500, 64, True)),
    (candidates.test_candidate_counts_around_the_register_sizes, (8, 2, 128, 65536, (1, 1500, 4500), 0, 1.0)),
    (candidates.test_candidate_counts_around_the_register_sizes, (16, 2, 64, 65537, (1000, 5000), 0, 4.0)),
    (candidates.test_candidate_counts_around_the_register_sizes, (16, 1, 64, 120001, (1000,), 0, 1.0)),
    (candidates.test_candidate_counts_around_the_register_sizes, (7, 1, 128, 65536, (1, 1500), 1, 1.0)),
    (runs.test_crowded_candidates, (16, 8, 64, 1, 40000, 0)),
    (runs.test_crowded_candidates, (32, 8, 64, 2, 40003, 1)),
    (heavy.test_planted_heavy_terms, (4, 128, 30017)),
    (heavy.test_planted_heavy_terms, (16, 64, 30017)),
    (heavy.test_terms_strewn_thin, (4, 128, 30017)),
    (chunks.test_filtered_rows_of_full_chunks, (4, 128)),
    (chunks.test_filtered_rows_of_full_chunks, (8, 64)),
    (parity.test_select_prefiltered_path, (24, 2, 128, 24000, 4, 64, 300)),
    (parity.test_prefilter_falls_back_when_all_scores_tie, ()),
    (parity.test_prefilter_falls_back_for_more_rows_than_a_gated_launch_has_row_blocks, ()),
    (parity.test_prefilter_with_one_token_carrying_most_of_the_mass, (True,)),
    (parity.test_prefilter_certifies_heavy_tailed_attention, (4.0, 0.4)),
    (parity.test_prefilter_certifies_model_like_attention, ()),
    (parity.test_prefilter_chunk_slots_overflow_into_the_row_pool, ()),
])
def test_workspace_of_the_prefiltered_path(ref, small, test, args):
    test(ref, *args)
    assert small and any(n < f for n, f in small)


@pytest.mark.parametrize("Hq,Hkv,d,L,W,k", [(32, 4, 64, 505, 400, 1), (32, 4, 64, 2500, 60, 9), (28, 4, 128, 20001, 64, 300), (24, 2, 64, 33001, 64, 200)])
@pytest.mark.parametrize("per_query", [False, True])
def test_calls_of_many_rows(Hq, Hkv, d, L, W, k, per_query):
    """Calls large enough for the pre-filtered path, of short rows too; every ninth row's keys are all equal."""
    import torch

    import paper_2503_08879_amd as sk

    S = 4
    P, G = (72 if L <= 8192 else 34) * 10 ** 6 // (4 * Hq * L), Hq // Hkv
    lists = G if per_query else 1
    n = S + lists * k + W
    g = torch.Generator(device="cuda")
    g.manual_seed(L)
    q = torch.randn((P, Hq, d), generator=g, device="cuda").bfloat16()
    K, V = (torch.randn((P, Hkv, L, d), generator=g, device="cuda", dtype=torch.bfloat16) for _ in range(2))
    flat = (torch.arange(P * Hkv, device="cuda") % 9 == 0).reshape(P, Hkv)
    K[flat] = K[flat][:, :1]
    desc = sk.select_desc(q, K, V, S, W, k, n, head_mode=int(per_query))
    ws = torch.empty(sk.sagekv_select_workspace_bytes(desc), dtype=torch.uint8, device="cuda")
    Kc = torch.zeros((P, Hkv, n, d), dtype=torch.bfloat16, device="cuda")
    Vc, kept = torch.zeros_like(Kc), torch.full((P, Hkv, n), -1, dtype=torch.int32, device="cuda")
    sk.sagekv_select(desc, q, K, V, Kc, Vc, kept, None, ws)
    assert sk.sagekv_select_redone_rows(desc, ws) == int(flat.sum())
    logits = torch.matmul(q.double().reshape(P, Hkv, G, d), K.double().transpose(2, 3).contiguous()) / d ** 0.5
    s = torch.softmax(logits, -1)
    s = s if per_query else s.sum(2, keepdim=True)
    top = torch.sort(torch.sort(s.float()[..., S:L - W], descending=True, stable=True).indices[..., :k], -1).values + S
    assert torch.equal(kept[..., S:S + lists * k].long(), top.reshape(P, Hkv, lists * k))
    at = kept.long().unsqueeze(-1).expand(P, Hkv, n, d)
    assert torch.equal(Kc, K.gather(2, at)) and torch.equal(Vc, V.gather(2, at))


def test_workspace_of_the_dense_path(ref, small):
    """fp32 rows in a workspace that only holds the logits and a score row: statistics, scores and selection in launches of their own."""
    q, K, V = parity.rand_case(4, 2, 4, 2, 64, 30000, F32)
    check(ref, F32, 0, q, K, V, 4, 64, 900)
    q, K, V = parity.rand_case(5, 1, 8, 2, 64, 26001, BF16)
    check(ref, BF16, 1, q, K, V, 4, 64, 900, flags=1)
