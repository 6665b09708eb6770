"""More rows (and lists, and chunks) to redo than the gated launches have workgroups: rows of equal keys, whose scores tie and whose
selection is the first k candidates, alone or between rows that the pre-filter certifies.  (As they are, these calls take the one-sweep path; test_gpu_filter_route has
them on the pre-filtered one.)"""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("every", [1, 2, 7])
@pytest.mark.parametrize("per_query", [False, True])
@pytest.mark.parametrize("L", [2500, 3073])
def test_many_rows_redone(every, per_query, L):
    import torch

    import paper_2503_08879_amd as sk

    P, Hq, Hkv, d, S, W, k = 80, 8, 4, 64, 4, 60, 40
    lists = Hq // Hkv if per_query else 1
    n = S + lists * k + W
    g = torch.Generator(device="cuda")
    g.manual_seed(L + every)
    q = torch.randn((P, Hq, d), generator=g, device="cuda").bfloat16()
    K, V = (torch.randn((P, Hkv, L, d), generator=g, device="cuda").bfloat16() for _ in range(2))
    flat = (torch.arange(P * Hkv, device="cuda") % every == 0).reshape(P, Hkv)
    K = torch.where(flat[..., None, None], K[:, :, :1], K)
    desc = sk.select_desc(q, K, V, S, W, k, n, head_mode=int(per_query))
    ws = torch.empty(sk.sagekv_select_workspace_bytes(desc), dtype=torch.uint8, device="cuda")
    Kc = torch.zeros((P, Hkv, n, d), dtype=torch.bfloat16, device="cuda")
    Vc = torch.zeros_like(Kc)
    kept = torch.full((P, Hkv, n), -1, dtype=torch.int32, device="cuda")
    for _ in range(2):
        sk.sagekv_select(desc, q, K, V, Kc, Vc, kept, None, ws)
    assert sk.sagekv_select_redone_rows(desc, ws) == int(flat.sum())
    logits = torch.matmul(q.double().reshape(P, Hkv, Hq // Hkv, d), K.double().transpose(2, 3).contiguous()) / d ** 0.5
    s = torch.softmax(logits, -1)
    s = s if per_query else s.sum(2, keepdim=True)
    cand = s.float()[..., S:L - W]
    top = torch.sort(torch.sort(cand, descending=True, stable=True).indices[..., :k], -1).values + S
    want = torch.cat([torch.arange(S, device="cuda").expand(P, Hkv, S), top.reshape(P, Hkv, lists * k),
                      torch.arange(L - W, L, device="cuda").expand(P, Hkv, W)], -1)
    assert torch.equal(kept.long(), want)
    at = want.unsqueeze(-1).expand(P, Hkv, n, d)
    assert torch.equal(Kc, K.gather(2, at)) and torch.equal(Vc, V.gather(2, at))
