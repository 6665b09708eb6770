"""The pre-filtered path's own tests on the pre-filtered path.  Calls of few rows take the one-sweep path when their workspace has room for it, and the
tests elsewhere are nearly all small; their count of redone rows means something else there.  Here they run once more with the least workspace, and
where that is room enough, with as many copies of the problems as make the call a large one.  Every call that the filter can serve must have gone through it:
the first word of the workspace then holds the number of redone rows, not the mark of the one-sweep path."""
import inspect
import itertools

import pytest

from tests import test_gpu_candidate_runs as runs
from tests import test_gpu_candidate_select as candidates
from tests import test_gpu_graph as graph
from tests import test_gpu_heavy_terms as heavy
from tests import test_gpu_many_redone as many
from tests import test_gpu_paged as paged
from tests import test_gpu_parity as parity
from tests import test_gpu_random_shapes as shapes
from tests import test_gpu_sample_edges as sample
from tests import test_gpu_score_chunks as chunks
from tests.test_gpu_shortlist import small  # noqa: F401 (fixture)

pytestmark = pytest.mark.gpu


def parameters(test):
    """The keyword arguments of every case of a parametrised test."""
    marks = [m for m in getattr(test, "pytestmark", []) if m.name == "parametrize"]
    for values in itertools.product(*(m.args[1] for m in marks)):
        args = {}
        for m, value in zip(marks, values):
            names = [n.strip() for n in m.args[0].split(",")]
            args.update(zip(names, value if len(names) > 1 else (value,)))
        yield args


TESTS = [
    heavy.test_planted_heavy_terms, heavy.test_terms_strewn_thin, runs.test_crowded_candidates,
    candidates.test_candidate_counts_around_the_register_sizes, sample.test_sample_edges, chunks.test_filtered_rows_of_full_chunks,
    many.test_many_rows_redone, paged.test_paged_prefiltered_bf16, paged.test_paged_G7_d64, paged.test_paged_per_query,
    parity.test_prefilter_with_one_token_carrying_most_of_the_mass, parity.test_prefilter_certifies_heavy_tailed_attention,
    parity.test_select_ranks_scores_below_the_normal_range_prefiltered, parity.test_layer_by_layer_on_two_streams_equals_one_batched_call,
    parity.test_prefiltered_select_is_deterministic, parity.test_select_prefiltered_path, parity.test_select_C2_shape_two_layers,
    parity.test_per_query_prefiltered_G7, graph.test_select_replayed_from_a_graph,
]
CASES = [(t, a) for t in TESTS for a in parameters(t)] + [
    (chunks.test_paged_rows_of_full_chunks, a) for a in parameters(chunks.test_paged_rows_of_full_chunks) if not a["want_scores"]] + [
    (paged.test_paged_select_with_peaked_attention, dict(page=16, want_scores=False, flags=0)),
    (parity.test_group_sum_order_when_few_tokens_hold_a_heads_mass, dict(route="prefiltered"))]
SHAPES = [(t, a) for t in (shapes.test_select_random_shape, shapes.test_select_paged_random_shape, shapes.test_per_query_random_shape)
          for a in parameters(t)]


def name(case):
    return "-".join([case[0].__name__[5:]] + [str(v) for v in case[1].values()]).replace(" ", "")


@pytest.fixture
def routes(small, monkeypatch):  # noqa: F811
    """Whether they went through the filtering pass: the calls without scores that it can serve."""
    import torch

    import paper_2503_08879_amd as sk

    seen, tables, counts = [], {}, {}
    make_pages, redone = sk.paged_select_desc, sk.sagekv_select_redone_rows

    def paged_select_desc(q, K, V, table, *args, **kw):
        desc, pages = make_pages(q, K, V, table, *args, **kw)
        tables[pages.block_table] = table
        return desc, pages

    def filtered(ws):
        return int(ws[:4].view(torch.int32)) >= 0

    def watch(call, paged):
        def watched(desc, *args):
            call(desc, *args)
            pages = args[:1] if paged else ()
            q, K, V, Kc, Vc, kept, scores, ws = args[len(pages):]
            counts.pop(ws.data_ptr(), None)
            if scores is not None or torch.cuda.is_current_stream_capturing() or redone(desc, ws) < 0:
                return
            if not filtered(ws):
                n = (72 if desc.L <= 8192 else 34) * 10 ** 6 // (4 * desc.n_problems * desc.n_q_heads * desc.L) + 1
                more = type(desc).from_buffer_copy(desc)
                more.n_problems *= n
                if paged:
                    table = tables[pages[0].block_table].repeat(n, 1)
                    pages = (type(pages[0]).from_buffer_copy(pages[0]),)
                    pages[0].block_table = table.data_ptr()
                else:
                    K, V = K.repeat(n, 1, 1, 1), V.repeat(n, 1, 1, 1)
                    more.k_stride_problem, more.k_stride_head, more.k_stride_token = K.stride()[:3]
                    more.v_stride_problem, more.v_stride_head, more.v_stride_token = V.stride()[:3]
                outs = [x.repeat(n, *[1] * (x.ndim - 1)) for x in (Kc, Vc, kept)]
                most = torch.empty(sk.sagekv_select_workspace_bytes(more), dtype=torch.uint8, device="cuda")
                call(more, *pages, q.repeat(n, 1, 1), K, V, *outs, None, most)
                counts[ws.data_ptr()], rest = divmod(redone(more, most), n)
                assert rest == 0
                for x, y in zip((Kc, Vc, kept), outs):
                    x.copy_(y[:len(x)])
                    assert torch.equal(y, x.repeat(n, *[1] * (x.ndim - 1)))
                ws = most
            seen.append(filtered(ws))
        return watched

    monkeypatch.setattr(sk, "paged_select_desc", paged_select_desc)
    monkeypatch.setattr(sk, "sagekv_select_redone_rows", lambda desc, ws: counts[ws.data_ptr()] if ws.data_ptr() in counts else redone(desc, ws))
    monkeypatch.setattr(sk, "sagekv_select", watch(sk.sagekv_select, False))
    monkeypatch.setattr(sk, "sagekv_select_paged", watch(sk.sagekv_select_paged, True))
    return seen


def run(ref, case):
    test, args = case
    test(**args, **({"ref": ref} if "ref" in inspect.signature(test).parameters else {}))


@pytest.mark.parametrize("case", CASES, ids=name)
def test_on_the_filtering_pass(ref, routes, case):
    run(ref, case)
    assert routes and all(routes), routes


@pytest.mark.parametrize("case", SHAPES, ids=name)
def test_random_shapes_on_the_filtering_pass(ref, routes, case):
    run(ref, case)  # (some shapes are the dense path's)
    assert all(routes), routes
