"""Decode steps over fp32 caches: every group size the kernel is compiled for and two launches of it, rows around a wave's block (16 or 32
tokens) and a workgroup's round of them, rows of many rounds, whole and sliced rows, pages, per-query rows, sink tokens under a query of their own, and in
the new token's place a value that is no number, which must leave with the step."""
import numpy as np
import pytest

import synth
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu
F32 = synth.F32


@pytest.mark.parametrize("G", [1, 2, 3, 4, 5, 6, 7, 8, 20])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("n,slot", [(2, 0), (15, 14), (17, 16), (33, 0), (129, 127), (193, 192), (257, 130), (385, 0), (700, 512), (1100, 1099)])
@pytest.mark.parametrize("layout", ["dense", "paged", "per_query", "window"])
def test_step(ref, G, d, n, slot, layout):
    import torch

    import paper_2503_08879_amd as sk

    P, Hkv, page = 2, 2, 16
    pq = layout == "per_query"
    S = min(3, n // 2) if pq or layout == "window" else 0
    k = (n - S) // (2 * G) if pq else 0
    W = n - S - (G * k if pq else 0)
    if slot < n - W:
        slot = n - W  # the window holds the new token
    rng = np.random.default_rng(n * 100 + G + d)
    draw = lambda *shape: rng.standard_normal(shape, dtype=np.float32)
    Kc, Vc, q, qs, kn, vn = draw(P, Hkv, n, d), draw(P, Hkv, n, d), draw(P, G * Hkv, d), draw(P, G * Hkv, d), draw(P, Hkv, d), draw(P, Hkv, d)
    Kd, Vd = torch.from_numpy(Kc).cuda(), torch.from_numpy(Vc).cuda()
    Kd[:, :, slot] = float("nan")
    Vd[:, :, slot] = float("inf")
    Kc[:, :, slot], Vc[:, :, slot] = kn, vn
    l = np.matmul(q.reshape(P, Hkv, G, d).astype(np.float64), Kc.astype(np.float64).transpose(0, 1, 3, 2)) / d ** 0.5
    if layout == "window" and S:
        l[..., :S] = np.matmul(qs.reshape(P, Hkv, G, d).astype(np.float64), Kc[:, :, :S].astype(np.float64).transpose(0, 1, 3, 2)) / d ** 0.5
    if pq:
        for g in range(G):
            for h in range(G):
                if h != g:
                    l[:, :, g, S + h * k:S + (h + 1) * k] = -np.inf
    w = np.exp(l - l.max(-1, keepdims=True))
    want = np.matmul(w / w.sum(-1, keepdims=True), Vc.astype(np.float64)).reshape(P, G * Hkv, d)
    desc, ws, out = gu.gpu_decode_setup(F32, P, G * Hkv, Hkv, d, S, k, W, n, head_mode=int(pq))
    at = slot - (n - W)
    ins = [torch.from_numpy(x).cuda() for x in (q, kn, vn)]
    state = torch.tensor([at, 0], dtype=torch.int32, device="cuda")
    if layout == "paged":
        per = (n + page - 1) // page
        pool = lambda X: torch.cat([X, X.new_full((P, Hkv, per * page - n, d), float("nan"))], 2).reshape(P, Hkv, per, page, d).transpose(1, 2).reshape(
            P * per, Hkv, page, d).contiguous()
        order = torch.randperm(P * per, device="cuda")
        Kp, Vp = (torch.empty_like(pool(X)).index_copy_(0, order, pool(X)) for X in (Kd, Vd))
        sk.sagekv_decode_step_paged(desc, sk.compact_pages(order.to(torch.int32).reshape(P, per), Kp, Vp), *ins, Kp, Vp, 0, state, out, ws)
        for X, new in ((Kp, kn), (Vp, vn)):
            got = X[order.reshape(P, per)[:, slot // page], :, slot % page]
            np.testing.assert_array_equal(got.cpu().numpy(), new)
    elif layout == "window":
        sk.sagekv_decode_step_window(desc, ins[0], torch.from_numpy(qs).cuda(), *ins[1:], Kd, Vd, at, out, ws)
    else:
        sk.sagekv_decode_step_ring(desc, *ins, Kd, Vd, state, out, ws)
    if layout != "window":
        assert state.tolist() == [at + 1, 0]
    if layout != "paged":
        np.testing.assert_array_equal(Kd.cpu().numpy(), Kc)
        np.testing.assert_array_equal(Vd.cpu().numpy(), Vc)
    gu.check_decode(out.cpu().numpy(), want, F32)


@pytest.mark.parametrize("rows,G,d,n,slot", [
    # a workgroup per row, many blocks per wave: rounds of 128 tokens (128 dims, or up to two heads) or 256
    (192, 1, 64, 600, 599), (192, 4, 64, 600, 555), (192, 7, 64, 600, 300), (192, 1, 128, 600, 470), (192, 4, 128, 600, 599), (192, 7, 128, 600, 580),
    (194, 1, 128, 2049, 2048), (194, 4, 128, 2049, 1500), (194, 7, 128, 2049, 2047), (194, 2, 64, 2049, 1030), (194, 4, 64, 2049, 1800), (194, 5, 64, 2049, 2048),
    # slices of several blocks per wave
    (100, 4, 64, 9000, 8999), (100, 7, 128, 9000, 4321), (64, 2, 128, 9000, 300), (150, 1, 128, 4001, 4000), (150, 5, 64, 4001, 1333), (190, 4, 128, 1999, 500),
    (6, 7, 128, 20011, 20010),
])
def test_rows_of_many_blocks(rows, G, d, n, slot):
    many_blocks(rows, G, d, n, slot, paged=False)


@pytest.mark.parametrize("rows,G,d,n,slot", [
    (192, 2, 64, 8203, 8202),   # 513 pages of 16, 8 waves: a wave asks for its 65th group's page
    (192, 4, 64, 8203, 8200),   # the same with blocks of two pages
    (192, 4, 128, 2049, 1999),
    (100, 7, 64, 2049, 1030),
])
def test_paged_rows_of_many_blocks(rows, G, d, n, slot):
    many_blocks(rows, G, d, n, slot, paged=True)


def many_blocks(rows, G, d, n, slot, paged):
    import torch

    import paper_2503_08879_amd as sk

    Hkv, page = 2, 16
    P, W = rows // Hkv, n - 17
    S, k, at = 0, n - W, slot - (n - W)  # a window that holds the new token's slot
    g = torch.Generator(device="cuda")
    g.manual_seed(n + G + d)
    draw = lambda *shape: torch.randn(shape, generator=g, device="cuda")
    q, kn, vn, K, V = draw(P, G * Hkv, d), draw(P, Hkv, d), draw(P, Hkv, d), draw(P, Hkv, n, d), draw(P, Hkv, n, d)
    # every wave's maximum grows from block to block in half of the heads, and falls in the others
    K += torch.linspace(-1, 1, n, device="cuda")[None, None, :, None] * q.reshape(P, Hkv, G, d).mean(2)[:, :, None]
    K[:, :, slot], V[:, :, slot] = float("nan"), float("inf")
    desc, ws, out = gu.gpu_decode_setup(F32, P, G * Hkv, Hkv, d, S, k, W, n)
    if paged:
        per = (n + page - 1) // page
        order = torch.randperm(P * per, device="cuda", generator=g)
        pools = []
        for X in (K, V):
            X = torch.cat([X, X.new_full((P, Hkv, per * page - n, d), float("nan"))], 2).reshape(P, Hkv, per, page, d).transpose(1, 2)
            pools.append(torch.empty((P * per, Hkv, page, d), device="cuda").index_copy_(0, order, X.reshape(P * per, Hkv, page, d)))
        table = order.to(torch.int32).reshape(P, per)
        sk.sagekv_decode_step_paged(desc, sk.compact_pages(table, *pools), q, kn, vn, *pools, at, None, out, ws)
    else:
        sk.sagekv_decode_step(desc, q, kn, vn, K, V, at, out, ws)
    K[:, :, slot], V[:, :, slot] = kn, vn
    l = torch.matmul(q.reshape(P, Hkv, G, d).double(), K.double().transpose(2, 3).contiguous()) / d ** 0.5
    want = torch.matmul(torch.softmax(l, -1), V.double()).reshape(P, G * Hkv, d)
    gu.check_decode(out.cpu().numpy(), want.cpu().numpy(), F32)
