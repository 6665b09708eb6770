"""Performance cases: what a program that uses this library has it do, through its public calls.

Eviction pass (once per prompt, after prefill): per layer as prefill produces the cache, or all layers in one
call; short prompts (the budget is a large share of the row) to 128K tokens; one top-k per KV head or one per
query head; strided and paged caches; bf16, and the small fp32 configuration.  Decoding (once per generated
token): all layers in one call, layer by layer in a recorded graph, per-query rows, pages, fp32.

Inputs: K, V, q ~ N(0, 1), needles along the queries' directions among the eviction candidates (key length 2 to 4,
as the synthetic caches of the benchmark have them) and sink tokens that hold some per cent of each head's mass.
"""
from __future__ import annotations

import math

import torch

import paper_2503_08879_amd as sk

DTYPES = {"bf16": torch.bfloat16, "f32": torch.float32}
NEEDLES = 64  # per row


def listed():
    def select(name, P, Hq, Hkv, d, L, S, W, k, dtype="bf16", mode="sum", layout="dense"):
        return dict(name=name, kind="select", P=P, Hq=Hq, Hkv=Hkv, d=d, L=L, S=S, W=W, k=k, dtype=dtype, mode=mode, layout=layout)

    def decode(name, P, Hq, Hkv, d, S, W, k, dtype="bf16", mode="sum", layout="dense", call="step"):
        return dict(name=name, kind="decode", P=P, Hq=Hq, Hkv=Hkv, d=d, S=S, W=W, k=k, dtype=dtype, mode=mode, layout=layout, call=call)

    return [
        # the tiny fp32 configuration: one layer, 4096 tokens, budget 256 (launches and latency)
        select("select_f32_tiny", 1, 4, 2, 64, 4096, 4, 64, 188, dtype="f32"),
        # one layer of a 32/8-head model as prefill finishes it, 32K and 128K tokens
        select("select_layer_32k", 1, 32, 8, 128, 32768, 4, 256, 1788),
        select("select_layer_128k", 1, 32, 8, 128, 131072, 4, 512, 3580),
        # a short prompt: the budget is a quarter of the row; all 32 layers in one call
        select("select_model_8k", 32, 32, 8, 128, 8192, 4, 256, 1788),
        # all 32 layers in one call, 32K and 128K tokens (the benchmark's workload)
        select("select_model_32k", 32, 32, 8, 128, 32768, 4, 256, 1788),
        select("select_model_128k", 32, 32, 8, 128, 131072, 4, 512, 3580),
        # one top-k per query head (the paper's literal rule, its split of an 8192-token budget), 28 layers of a 28/4-head model
        select("select_per_query_128k", 28, 28, 4, 128, 131072, 2048, 2560, 512, mode="pq"),
        # a serving engine's paged cache (pages of 16 tokens), a batch of 16 sequences of one layer, ragged length, into pages
        select("select_paged_batch", 16, 28, 4, 128, 40013, 4, 128, 892, layout="paged"),
        # the tiny fp32 configuration, one decode step
        decode("decode_f32_tiny", 1, 4, 2, 64, 4, 64, 188, dtype="f32"),
        # one generated token, layer by layer as a model needs it: a recorded graph of 32 one-layer steps
        decode("decode_token_layers", 32, 32, 8, 128, 4, 512, 3580, call="graph"),
        # one step over all 32 layers in one call (the benchmark's workload)
        decode("decode_model_4k", 32, 32, 8, 128, 4, 512, 3580),
        # per-query rows of 8192 tokens in pages, 28 layers x 4 sequences
        decode("decode_per_query_paged", 112, 28, 4, 128, 2048, 2560, 512, mode="pq", layout="paged"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _paper_split(B, G):
    share, p = B // (2 * G), 1
    while p <= share // 2:
        p *= 2
    return B // 4, B - B // 4 - G * p, p  # sink, recent, k


def draw(rng):
    Hq, Hkv, d = rng.choice([(32, 8, 128), (32, 8, 128), (28, 4, 128), (28, 4, 128), (8, 2, 64)])
    G = Hq // Hkv
    dtype = "f32" if rng.random() < 0.15 else "bf16"
    eb = 4 if dtype == "f32" else 2
    mode = "pq" if rng.random() < 0.25 else "sum"
    layout = "paged" if rng.random() < 0.25 else "dense"
    if rng.random() < 0.6:
        L = _log_int(rng, 2048, 262144 if dtype == "bf16" else 32768)
        B = min(_log_int(rng, 512, 8192), L // 2)
        if mode == "pq":
            S, W, k = _paper_split(B, G)
        else:
            S, W = rng.choice([1, 4, 4, 64]), max(1, B // rng.randint(6, 12))
            k = B - S - W
        most = (1 << 32 if dtype == "bf16" else 1 << 30) // (Hkv * L * d * eb)  # K of at most 4 GiB (fp32: 1 GiB)
        P = 1 if rng.random() < 0.4 else _log_int(rng, 1, max(1, min(32, most)))
        return dict(kind="select", P=P, Hq=Hq, Hkv=Hkv, d=d, L=L, S=S, W=W, k=k, dtype=dtype, mode=mode, layout=layout)
    B = _log_int(rng, 256, 8192)
    if mode == "pq":
        S, W, k = _paper_split(B, G)
    else:
        S, W = rng.choice([1, 4, 4, 64]), max(1, B // rng.randint(6, 12))
        k = B - S - W
    P = rng.choice([1, 2, _log_int(rng, 2, 128), 32])
    call = "graph" if layout == "dense" and P <= 32 and rng.random() < 0.4 else "step"
    return dict(kind="decode", P=P, Hq=Hq, Hkv=Hkv, d=d, S=S, W=W, k=k, dtype=dtype, mode=mode, layout=layout, call=call)


PAGE = 16
APPENDED = 37  # tokens a "step" case's cache has taken in before the measured one


def _lists(c):
    return c["Hq"] // c["Hkv"] if c["mode"] == "pq" else 1


def _row_len(c):
    return c["S"] + _lists(c) * c["k"] + c["W"]


def _head_mode(c):
    return sk.PER_QUERY if c["mode"] == "pq" else sk.GROUP_SUM


def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _table(gen, P, tokens):
    """A shuffled block table for P problems of `tokens` tokens, and the number of pages."""
    per = (tokens + PAGE - 1) // PAGE
    return torch.randperm(P * per, generator=gen, device="cuda").to(torch.int32).reshape(P, per), P * per


def _select_inputs(c, seed):
    """q [P, Hq, d]; K, V dense [P, Hkv, L, d] or pools [pages, Hkv, PAGE, d]; block table or None."""
    gen, t = _generator(seed), DTYPES[c["dtype"]]
    P, Hq, Hkv, d, L, S, W = (c[n] for n in ("P", "Hq", "Hkv", "d", "L", "S", "W"))
    G, E = Hq // Hkv, L - S - W
    q = torch.randn((P, Hq, d), generator=gen, device="cuda").to(t)
    n = min(NEEDLES, E)
    unit = torch.nn.functional.normalize(q.float(), dim=-1).reshape(P, Hkv, G, d)
    step = E // n
    pos = S + torch.arange(n, device="cuda") * step + torch.randint(0, step, (P, Hkv, n), generator=gen, device="cuda")
    head = (torch.arange(n, device="cuda") % G).reshape(1, 1, n, 1).expand(P, Hkv, n, d)
    length = 2.0 + 2.0 * torch.rand((P, Hkv, n, 1), generator=gen, device="cuda")
    needles = length * torch.gather(unit, 2, head) + 0.1 * torch.randn((P, Hkv, n, d), generator=gen, device="cuda")
    n_s = min(S, 4)
    sinks = 8.0 * unit.sum(2, keepdim=True) + 0.1 * torch.randn((P, Hkv, n_s, d), generator=gen, device="cuda")
    pos = torch.cat([torch.arange(n_s, device="cuda").expand(P, Hkv, n_s), pos], 2)
    rows = torch.cat([sinks, needles], 2).to(t)
    p_at = torch.arange(P, device="cuda").reshape(P, 1, 1)
    c_at = torch.arange(Hkv, device="cuda").reshape(1, Hkv, 1)
    if c["layout"] == "paged":
        table, pages = _table(gen, P, L)
        K = torch.randn((pages, Hkv, PAGE, d), generator=gen, device="cuda", dtype=t)
        V = torch.randn((pages, Hkv, PAGE, d), generator=gen, device="cuda", dtype=t)
        K[table.long()[p_at, pos // PAGE], c_at, pos % PAGE] = rows
        return q, K, V, table
    K = torch.randn((P, Hkv, L, d), generator=gen, device="cuda", dtype=t)
    V = torch.randn((P, Hkv, L, d), generator=gen, device="cuda", dtype=t)
    K[p_at, c_at, pos] = rows
    return q, K, V, None


def _decode_inputs(c, seed):
    """q [P, Hq, d]; k_new, v_new [P, Hkv, d]; the reduced cache dense [P, Hkv, len, d] or pools; block table or None."""
    gen, t = _generator(seed), DTYPES[c["dtype"]]
    P, Hq, Hkv, d, n = c["P"], c["Hq"], c["Hkv"], c["d"], _row_len(c)
    q, kn, vn = (torch.randn((P, h, d), generator=gen, device="cuda").to(t) for h in (Hq, Hkv, Hkv))
    table, shape = None, (P, Hkv, n, d)
    if c["layout"] == "paged":
        table, pages = _table(gen, P, n)
        shape = (pages, Hkv, PAGE, d)
    Kc = torch.randn(shape, generator=gen, device="cuda", dtype=t)
    Vc = torch.randn(shape, generator=gen, device="cuda", dtype=t)
    return q, kn, vn, Kc, Vc, table


def _out_pages(c, seed):
    return _table(_generator(seed + 1), c["P"], _row_len(c))


def prepare(case, seed):
    c = case
    P, Hq, Hkv, d, S, W, k, n = c["P"], c["Hq"], c["Hkv"], c["d"], c["S"], c["W"], c["k"], _row_len(c)
    if c["kind"] == "select":
        q, K, V, table = _select_inputs(c, seed)
        s = dict(case=c, q=q, K=K, V=V, table=table, kept=torch.zeros((P, Hkv, n), dtype=torch.int32, device="cuda"))
        if table is None:
            s["desc"] = sk.select_desc(q, K, V, S, W, k, n, head_mode=_head_mode(c))
            s["Kc"] = torch.zeros((P, Hkv, n, d), dtype=K.dtype, device="cuda")
            s["Vc"] = torch.zeros_like(s["Kc"])
        else:
            s["desc"], s["pages"] = sk.paged_select_desc(q, K, V, table, c["L"], S, W, k, n, head_mode=_head_mode(c))
            s["out_table"], pages = _out_pages(c, seed)
            s["Kc"] = torch.zeros((pages, Hkv, PAGE, d), dtype=K.dtype, device="cuda")
            s["Vc"] = torch.zeros_like(s["Kc"])
            s["out_pages"] = sk.compact_pages(s["out_table"], s["Kc"], s["Vc"])
        s["ws"] = torch.empty(sk.sagekv_select_workspace_bytes(s["desc"]), dtype=torch.uint8, device="cuda")
        return s
    q, kn, vn, Kc, Vc, table = _decode_inputs(c, seed)
    s = dict(case=c, q=q, kn=kn, vn=vn, Kc=Kc, Vc=Vc, table=table, out=torch.zeros((P, Hq, d), device="cuda"))
    dt = sk.F32 if c["dtype"] == "f32" else sk.BF16
    per_call = 1 if c["call"] == "graph" else P
    s["desc"] = sk.decode_desc(per_call, Hq, Hkv, d, dt, S, k, W, n, head_mode=_head_mode(c))
    s["ws"] = torch.empty(max(16, sk.sagekv_decode_workspace_bytes(s["desc"])), dtype=torch.uint8, device="cuda")
    if table is not None:
        s["pages"] = sk.compact_pages(table, Kc, Vc)
    if c["call"] == "graph":  # one recorded step per layer, the append counts on the device
        s["rings"] = torch.zeros((P, 2), dtype=torch.int32, device="cuda")
        sk.sagekv_decode_attn(s["desc"], q[0], Kc[0], Vc[0], n, s["out"][0], s["ws"])
        torch.cuda.synchronize()
        s["graph"] = torch.cuda.CUDAGraph()
        with torch.cuda.graph(s["graph"]):
            for p in range(P):
                sk.sagekv_decode_step_ring(s["desc"], q[p], kn[p], vn[p], Kc[p], Vc[p], s["rings"][p], s["out"][p], s["ws"])
    return s


def run(state):
    s = state
    c = s["case"]
    if c["kind"] == "select":
        if s["table"] is None:
            sk.sagekv_select(s["desc"], s["q"], s["K"], s["V"], s["Kc"], s["Vc"], s["kept"], None, s["ws"])
        else:
            sk.sagekv_select_into_pages(s["desc"], s["pages"], s["out_pages"], s["q"], s["K"], s["V"], s["Kc"], s["Vc"],
                                        s["kept"], None, s["ws"])
        return {"kept": s["kept"], "Kc": s["Kc"], "Vc": s["Vc"]}
    if c["call"] == "graph":
        s["graph"].replay()
    elif s["table"] is None:
        sk.sagekv_decode_step(s["desc"], s["q"], s["kn"], s["vn"], s["Kc"], s["Vc"], APPENDED, s["out"], s["ws"])
    else:
        sk.sagekv_decode_step_paged(s["desc"], s["pages"], s["q"], s["kn"], s["vn"], s["Kc"], s["Vc"], APPENDED, None,
                                    s["out"], s["ws"])
    return {"out": s["out"], "Kc": s["Kc"], "Vc": s["Vc"]}


def work(case):
    c = case
    rows, d, n, eb = c["P"] * c["Hkv"], c["d"], _row_len(c), 4 if c["dtype"] == "f32" else 2
    if c["kind"] == "select":
        # K read once; of the survivors V is read, K and V are written, and their positions
        return {"bytes": rows * (c["L"] * d * eb + 3 * n * d * eb + 4 * n), "flops": 2 * c["P"] * c["Hq"] * c["L"] * d}
    attended = c["S"] + c["k"] + c["W"]  # per query head
    return {"bytes": rows * (2 * n * d * eb + 4 * d * eb) + c["P"] * c["Hq"] * d * (eb + 4), "flops": 4 * c["P"] * c["Hq"] * attended * d}


def tolerance(case):
    # kept sets and gathered rows are those of the fp64 definition, bit for bit
    if case["kind"] == "select":
        return "exact"
    # fp32 sums; with bf16 caches the softmax weights of some shapes are rounded to bf16, as the values are
    return {"rel": 2e-6} if case["dtype"] == "f32" else {"rel": 6e-3, "max": 0.05}


def _row_of(pool, table, p, h, tokens):
    """Tokens [0, tokens) of problem p, KV head h of a paged cache."""
    return pool[table[p].long(), h].reshape(-1, pool.shape[-1])[:tokens]


def _exact_select(c, seed):
    q, K, V, table = _select_inputs(c, seed)
    P, Hq, Hkv, d, L, S, W, k, n = c["P"], c["Hq"], c["Hkv"], c["d"], c["L"], c["S"], c["W"], c["k"], _row_len(c)
    G = Hq // Hkv
    kept = torch.zeros((P, Hkv, n), dtype=torch.int32, device="cuda")
    if table is None:
        Kc = torch.zeros((P, Hkv, n, d), dtype=K.dtype, device="cuda")
    else:
        out_table, pages = _out_pages(c, seed)
        Kc = torch.zeros((pages, Hkv, PAGE, d), dtype=K.dtype, device="cuda")
    Vc = torch.zeros_like(Kc)
    t = torch.arange(n, device="cuda")
    for p in range(P):
        for h in range(Hkv):
            Kr, Vr = (K[p, h], V[p, h]) if table is None else (_row_of(K, table, p, h, L), _row_of(V, table, p, h, L))
            logits = torch.mm(q[p, h * G:(h + 1) * G].double(), Kr.double().t().contiguous()) / math.sqrt(d)
            prob = torch.softmax(logits, dim=1)
            lists = prob if c["mode"] == "pq" else prob.sum(0, keepdim=True)
            parts = [torch.arange(S, device="cuda")]
            for s in lists.float():  # ranked as fp32 values, equal ones by position
                order = torch.sort(s[S:L - W], descending=True, stable=True).indices[:k]
                parts.append(S + torch.sort(order).values)
            idx = torch.cat(parts + [torch.arange(L - W, L, device="cuda")])
            kept[p, h] = idx.to(torch.int32)
            if table is None:
                Kc[p, h], Vc[p, h] = Kr[idx], Vr[idx]
            else:
                page = out_table[p].long()[t // PAGE]
                Kc[page, h, t % PAGE], Vc[page, h, t % PAGE] = Kr[idx], Vr[idx]
    return {"kept": kept, "Kc": Kc, "Vc": Vc}


def _exact_decode(c, seed):
    q, kn, vn, Kc, Vc, table = _decode_inputs(c, seed)
    P, Hq, Hkv, d, S, W, k, n = c["P"], c["Hq"], c["Hkv"], c["d"], c["S"], c["W"], c["k"], _row_len(c)
    G = Hq // Hkv
    slot = S + _lists(c) * k + (0 if c["call"] == "graph" else APPENDED % W)
    if table is None:
        Kc[:, :, slot], Vc[:, :, slot] = kn, vn
    else:
        page = table.long()[:, slot // PAGE]
        Kc[page, :, slot % PAGE], Vc[page, :, slot % PAGE] = kn, vn
    out = torch.zeros((P, Hq, d), dtype=torch.float64, device="cuda")
    t = torch.arange(n, device="cuda")
    for p in range(P):
        for h in range(Hkv):
            Kr, Vr = (Kc[p, h], Vc[p, h]) if table is None else (_row_of(Kc, table, p, h, n), _row_of(Vc, table, p, h, n))
            logits = torch.mm(q[p, h * G:(h + 1) * G].double(), Kr.double().t().contiguous()) / math.sqrt(d)
            if c["mode"] == "pq":
                own = (t - S).div(k, rounding_mode="floor").reshape(1, n) == torch.arange(G, device="cuda").reshape(G, 1)
                common = (t < S) | (t >= S + G * k)
                logits = torch.where(own & ~common | common, logits, torch.full_like(logits, -math.inf))
            out[p, h * G:(h + 1) * G] = torch.mm(torch.softmax(logits, dim=1), Vr.double())
    return {"out": out, "Kc": Kc, "Vc": Vc}


def exact(case, seed):
    return _exact_select(case, seed) if case["kind"] == "select" else _exact_decode(case, seed)
