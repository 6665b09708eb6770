"""The gather on both sides of the size from which it stores nontemporally: rows, byte for byte, at the pass's own kept positions."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,d", [("bf16", 64), ("bf16", 128), ("f32", 64), ("f32", 128)])
@pytest.mark.parametrize("pages", [False, True])
@pytest.mark.parametrize("megabytes", [90, 97])  # the line is at 96
def test_gathered_rows(dtype, d, pages, megabytes):
    import torch

    import paper_2503_08879_amd as sk

    t = torch.bfloat16 if dtype == "bf16" else torch.float32
    P, Hkv, S, W = 3, 5, 4, 65
    n = (megabytes << 20) // (2 * P * Hkv * d * t.itemsize) + 1
    L, k = n + 123, n - S - W
    g = torch.Generator(device="cuda")
    g.manual_seed(megabytes + d)
    q = torch.randn((P, 2 * Hkv, d), generator=g, device="cuda").to(t)
    K, V = (torch.randn((P, Hkv, L, d), generator=g, device="cuda").to(t) for _ in range(2))
    desc = sk.select_desc(q, K, V, S, W, k, n)
    ws = torch.empty(sk.sagekv_select_workspace_bytes(desc), dtype=torch.uint8, device="cuda")
    kept = torch.full((P, Hkv, n), -1, dtype=torch.int32, device="cuda")
    if pages:
        per = -(-n // 16)
        table = torch.randperm(P * per, generator=g, device="cuda").to(torch.int32).reshape(P, per)
        Kc = torch.zeros((P * per, Hkv, 16, d), dtype=t, device="cuda")
        Vc = torch.zeros_like(Kc)
        sk.sagekv_select_into_pages(desc, None, sk.compact_pages(table, Kc, Vc), q, K, V, Kc, Vc, kept, None, ws)
        Kc, Vc = (x[table.long()].transpose(1, 2).reshape(P, Hkv, per * 16, d)[:, :, :n] for x in (Kc, Vc))
    else:
        Kc = torch.zeros((P, Hkv, n, d), dtype=t, device="cuda")
        Vc = torch.zeros_like(Kc)
        sk.sagekv_select(desc, q, K, V, Kc, Vc, kept, None, ws)
    assert bool((kept[..., 1:] > kept[..., :-1]).all())
    at = kept.long().unsqueeze(-1).expand(P, Hkv, n, d)
    assert torch.equal(Kc, K.gather(2, at)) and torch.equal(Vc, V.gather(2, at))
