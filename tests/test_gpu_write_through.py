"""Calls on both sides of the size (1 GiB of keys) from which the filtering pass writes its candidate records through L2: the same
kept sets as the one-sweep dense path's."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Hq,per_query", [(32, 0), (56, 0), (56, 1), (96, 0)])
@pytest.mark.parametrize("L", [65536, 65537])  # 128 rows x 65536 x 64 x 2 bytes: 1 GiB
def test_both_sides(Hq, per_query, L):
    import torch

    import paper_2503_08879_amd as sk

    P, Hkv, d, S, W = 16, 8, 64, 4, 64
    k = 600 // (Hq // Hkv if per_query else 1)
    n = S + (Hq // Hkv if per_query else 1) * k + W
    g = torch.Generator(device="cuda")
    g.manual_seed(L + Hq)
    q = torch.randn((P, Hq, d), generator=g, device="cuda").bfloat16()
    K, V = (torch.randn((P, Hkv, L, d), generator=g, device="cuda", dtype=torch.bfloat16) for _ in range(2))
    K[:, :, 5000:5700] += 0.5 * q.reshape(P, Hkv, -1, d).float().mean(2, keepdim=True).bfloat16()  # a crowd: several runs per wave
    got = []
    for flags in (0, sk.SELECT_DENSE):
        desc = sk.select_desc(q, K, V, S, W, k, n, head_mode=per_query, flags=flags)
        ws = torch.empty(sk.sagekv_select_workspace_bytes(desc), dtype=torch.uint8, device="cuda")
        Kc = torch.zeros((P, Hkv, n, d), dtype=torch.bfloat16, device="cuda")
        kept = torch.full((P, Hkv, n), -1, dtype=torch.int32, device="cuda")
        sk.sagekv_select(desc, q, K, V, Kc, torch.zeros_like(Kc), kept, None, ws)
        assert sk.sagekv_select_redone_rows(desc, ws) == (-1 if flags else 0)
        got.append(kept)
    assert torch.equal(got[0], got[1])
