"""GPU parity of small decode batches: few rows of many partials (a merge
workgroup per row) and the short key chunks that leave a small batch enough
items, against the oracle."""

import numpy as np
import pytest
import torch

from gpu_helpers import assert_parity, oracle_for, run_library, to_device
from paper_2509_02121_amd import halo
from gpu_helpers import params_of
from workloads import build_workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,d,out_dtype", [(torch.bfloat16, 128, torch.bfloat16), (torch.bfloat16, 64, torch.bfloat16),
                                               (torch.bfloat16, 128, torch.float32), (torch.float32, 128, torch.float32),
                                               (torch.float32, 64, torch.float32)])
@pytest.mark.parametrize("keys", [520, 1088, 9000, 17000])
def test_few_rows_of_many_partials(gpu_lib, dtype, d, out_dtype, keys):
    """9 partials (one more than the fixed slots), as many as a row's groups of
    threads take in one round and more, one request without private keys, and
    one without any key beside them."""
    print(f"case: many partials {dtype} d{d} {out_dtype} {keys} keys", flush=True)
    seg_len = [70, keys, keys // 2 + 3]
    paths = [[0, 1], [0, 2], [0], []]
    w = build_workload("parts", 81, 6, 2, d, dtype, seg_len, paths, value_scale=0.5 if dtype == torch.bfloat16 else 1.0)
    o, lse, pa = run_library(w, out_dtype)
    m = pa.plan.inspect()
    assert np.diff(m["merge_indptr"]).max() > 8
    ro, rl, rows = oracle_for(w)
    assert_parity(w, o, lse, ro, rl, rows, f"{keys} keys")


@pytest.mark.parametrize("n_req,prefix,private,longest", [(1, 0, 500, 64), (4, 1000, 200, 64), (16, 2000, 170, 96),
                                                          (32, 2000, 170, 256), (64, 2048, 290, 512)])
def test_chunk_lengths_of_small_batches(gpu_lib, n_req, prefix, private, longest):
    """The planner's key chunks shorten as the batch gets smaller (longest:
    keys of the longest chunk), fresh and after growing in place."""
    print(f"case: chunk lengths {n_req} requests", flush=True)
    rng = np.random.default_rng(n_req)
    own = [int(x) for x in rng.integers(private * 3 // 4, private * 5 // 4, size=n_req)]
    seg_len = ([prefix] if prefix else []) + own
    paths = [([0] if prefix else []) + [len(seg_len) - n_req + r] for r in range(n_req)]
    w = build_workload("chunks", 82, 32, 8, 128, torch.bfloat16, seg_len, paths, value_scale=0.5)
    o, lse, pa = run_library(w)
    spans = pa.plan.inspect()["spans"]
    assert (spans[:, 2] - spans[:, 1]).max() == longest
    sample = list(range(0, n_req, max(1, n_req // 4)))
    ro, rl, rows = oracle_for(w, sample)
    assert_parity(w, o, lse, ro, rl, rows, "fresh")
    # the plan of a shorter batch, grown in place to this one
    grown = w.forest_csr()
    short = {k: v.copy() for k, v in grown.items() if v is not None}
    cut = np.array([0] * (1 if prefix else 0) + [int(rng.integers(0, 60)) for _ in own], np.int32)
    short["seg_len"] = grown["seg_len"] - cut
    pages = [w.seg_pages[s][:(int(n) + 15) // 16] for s, n in enumerate(short["seg_len"])]
    short["seg_page_indptr"] = np.concatenate([[0], np.cumsum([len(p) for p in pages])]).astype(np.int32)
    short["seg_page_ids"] = np.concatenate(pages).astype(np.int32)
    pa = halo.PrefixAttention(params_of(w), short, "cuda")
    assert pa.update(grown)
    o, lse = pa.run(w.q, w.k_pool, w.v_pool)
    torch.cuda.synchronize()
    assert_parity(w, o.double().cpu().numpy(), lse.double().cpu().numpy(), ro, rl, rows, "grown")


@pytest.mark.parametrize("keys", [300, 900, 9000])
@pytest.mark.parametrize("where", ["q", "k", "v"])
def test_nan_inputs_stay_visible_through_the_merge(gpu_lib, keys, where):
    """A NaN in a query, a key or a value reaches exactly the outputs it
    belongs to, however many partials (a few, more than 8, many) a row has."""
    print(f"case: NaN in {where}, {keys} private keys", flush=True)
    w = to_device(build_workload("nan", 83, 8, 2, 128, torch.bfloat16, [keys, keys - 7], [[0], [1]], value_scale=0.5))
    page = int(w.seg_pages[0][3])
    hit = np.zeros((2, 8, 128), bool)
    if where == "q":
        w.q[0, 0, 5] = float("nan")
        hit[0, 0] = True
    elif where == "k":
        w.k_pool[page, 0, 2, 7, 3] = float("nan")
        hit[0, :4] = True
    else:
        w.v_pool[page, 0, 9, 4] = float("nan")
        hit[0, :4, 9] = True
    pa = halo.PrefixAttention(params_of(w), w.forest_csr(), "cuda")
    assert pa.plan.stats()["num_partial_rows"] > 0
    o, lse = pa.run(w.q, w.k_pool, w.v_pool)
    assert (torch.isnan(o).cpu().numpy() == hit).all()
    # rows with NaN scores have LSE -inf, however they were split
    assert (torch.isneginf(lse).cpu().numpy() == (hit.all(axis=2) if where != "v" else False)).all()


def test_decodes_on_two_streams_have_a_workspace_each(gpu_lib):
    """Calls of one object on two streams, each with its own queries, write
    their partials to different workspaces, and to a third while captured."""
    print("case: small decode on two streams", flush=True)
    w = to_device(build_workload("two streams", 84, 8, 2, 128, torch.bfloat16, [300, 350], [[0], [1]],
                                 value_scale=0.5))
    pa = halo.PrefixAttention(params_of(w), w.forest_csr(), "cuda")
    assert pa.plan.workspace_bytes > 0
    streams = [torch.cuda.Stream() for _ in range(2)]
    qs = [w.q * x for x in (1.0, -2.0, 0.5)]
    want = [pa.run(q, w.k_pool, w.v_pool) for q in qs]
    torch.cuda.synchronize()
    used = set()
    lib_run = halo.prefix_attn_decode

    def spy(plan, meta, q, k, v, o, lse, workspace, stream=None):
        used.add(workspace.data_ptr())
        lib_run(plan, meta, q, k, v, o, lse, workspace, stream)

    halo.prefix_attn_decode = spy
    try:
        got = [pa.alloc_outputs(q) for q in qs]
        torch.cuda.synchronize()
        for _ in range(20):
            for q, out, s in zip(qs, got, streams):
                pa.run(q, w.k_pool, w.v_pool, *out, stream=s)
        torch.cuda.synchronize()
        assert len(used) == 2
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=streams[0]):
            pa.run(qs[2], w.k_pool, w.v_pool, *got[2])
        assert len(used) == 3
    finally:
        halo.prefix_attn_decode = lib_run
    for _ in range(3):
        for q, out, s in zip(qs, got, streams):
            pa.run(q, w.k_pool, w.v_pool, *out, stream=s)
        graph.replay()
        torch.cuda.synchronize()
        for (o, lse), (wo, wl) in zip(got, want):
            assert torch.equal(o, wo) and torch.equal(lse, wl)


def test_workspaces_of_many_streams_are_bounded(gpu_lib):
    print("case: workspaces of many streams", flush=True)
    w = to_device(build_workload("streams", 85, 8, 2, 128, torch.bfloat16, [300, 350], [[0], [1]], value_scale=0.5))
    pa = halo.PrefixAttention(params_of(w), w.forest_csr(), "cuda")
    want, _ = pa.run(w.q, w.k_pool, w.v_pool)
    torch.cuda.synchronize()
    outs = [pa.run(w.q, w.k_pool, w.v_pool, stream=torch.cuda.Stream())[0] for _ in range(pa.MAX_WORKSPACES + 8)]
    torch.cuda.synchronize()
    assert len(pa._ws) <= pa.MAX_WORKSPACES
    assert all(torch.equal(o, want) for o in outs)


def test_a_call_bound_during_a_capture_runs_eagerly_too(gpu_lib):
    """Bound while a stream is captured: the graph replays, and eager calls of
    the same callable leave the graph's memory alone."""
    print("case: bound during a capture", flush=True)
    w = to_device(build_workload("bound", 86, 8, 2, 128, torch.bfloat16, [300, 350], [[0], [1]], value_scale=0.5))
    pa = halo.PrefixAttention(params_of(w), w.forest_csr(), "cuda")
    stream, side = torch.cuda.Stream(), torch.cuda.Stream()
    want, want_lse = pa.run(w.q, w.k_pool, w.v_pool, stream=stream)
    o, lse = pa.alloc_outputs(w.q)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        call = pa.bind(w.q, w.k_pool, w.v_pool, o, lse, stream)
        call()
    for _ in range(3):
        for again in (graph.replay, call):
            o.zero_()
            torch.cuda.synchronize()
            with torch.cuda.stream(side):
                again()
            torch.cuda.synchronize()
            assert torch.equal(o, want) and torch.equal(lse, want_lse)
