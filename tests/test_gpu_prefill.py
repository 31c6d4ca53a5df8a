"""GPU parity of chunked prefill (§4.1, prefix caching) at the sizes where its
work lists change: row blocks of 32 rows per wave and 128 (or 256) per
workgroup, against the oracle."""

import pytest
import torch

import numpy as np
from gpu_helpers import assert_parity, oracle_for, params_of, to_device
from paper_2509_02121_amd import halo
from workloads import build_workload

pytestmark = pytest.mark.gpu


def _run(w, options=None, out_dtype=None):
    to_device(w)
    pa = halo.PrefixAttention(params_of(w, out_dtype), w.forest_csr(), "cuda", options)
    o, lse = pa.run(w.q, w.k_pool, w.v_pool)
    torch.cuda.synchronize()
    return o.double().cpu().numpy(), lse.double().cpu().numpy(), pa


@pytest.mark.parametrize("options", [None, {"wide_rows": 32}, {"wide_rows": 256}],
                         ids=["128rows", "32rows", "256rows"])
@pytest.mark.parametrize("d,out_dtype", [(64, torch.float32), (128, torch.bfloat16), (128, torch.float32)])
def test_row_blocks_of_prefill_items(gpu_lib, d, out_dtype, options):
    """Chunks that end just before, at and after a wave's 32 rows, a
    workgroup's 128 and 256, over cached segments that end inside a page, a
    step and a span, in workgroups of four and of eight waves."""
    print(f"case: prefill row blocks d{d} {out_dtype} {options}", flush=True)
    q_len = [1, 31, 32, 33, 127, 128, 129, 255, 257]
    seg_len = [0, 5, 48, 1023, 1025] + q_len
    paths = [[i % 5, 5 + i] if i else [5] for i in range(len(q_len))]
    w = build_workload("rowblocks", 71, 3, 3, d, torch.bfloat16, seg_len, paths, q_len, value_scale=0.5)
    o, lse, _ = _run(w, options, out_dtype)
    ro, rl, rows = oracle_for(w)
    assert_parity(w, o, lse, ro, rl, rows, f"row blocks d{d} {options}")
    assert np.isfinite(o).all()


@pytest.mark.parametrize("dtype,d,out_dtype", [(torch.bfloat16, 128, torch.bfloat16), (torch.bfloat16, 64, torch.float32),
                                               (torch.float32, 128, torch.float32), (torch.float32, 64, torch.float32)])
@pytest.mark.parametrize("prefix,q_len", [(3001, [70]), (1500, [1, 200, 33]), (0, [900]), (7000, [1])])
def test_items_cut_into_pieces(gpu_lib, dtype, d, out_dtype, prefix, q_len):
    """Few items with many keys: their keys are cut into pieces (inside cached
    segments and inside the causal chunk, where some rows of a piece see no
    key) and merged; without the workspace the items run uncut."""
    print(f"case: prefill pieces {dtype} d{d} prefix {prefix} chunks {q_len}", flush=True)
    seg_len = [prefix // 3, prefix - prefix // 3] + q_len
    paths = [[0, 1, 2 + i] for i in range(len(q_len))]
    w = build_workload("pieces", 72, 6, 2, d, dtype, seg_len, paths, q_len,
                       value_scale=0.5 if dtype == torch.bfloat16 else 1.0)
    o, lse, pa = _run(w, None, out_dtype)
    assert pa.plan.workspace_bytes > 0 and pa.plan.stats()["num_merge_rows"] > 0, "the items are cut"
    ro, rl, rows = oracle_for(w)
    assert_parity(w, o, lse, ro, rl, rows, "pieces")
    o2, lse2 = pa.alloc_outputs(w.q)
    halo.prefix_attn_prefill(pa.plan, pa.meta, w.q, w.k_pool, w.v_pool, o2, lse2, None)
    torch.cuda.synchronize()
    assert_parity(w, o2.double().cpu().numpy(), lse2.double().cpu().numpy(), ro, rl, rows, "uncut")


def test_piecewise_prefill_on_two_streams_and_in_a_graph(gpu_lib):
    """Calls of one object that overlap on two streams have a workspace each,
    and a captured call replays with the eager call's bits."""
    print("case: prefill pieces on two streams, captured", flush=True)
    w = to_device(build_workload("streams", 73, 8, 2, 128, torch.bfloat16, [5000, 150], [[0, 1]], [150],
                                 value_scale=0.5))
    pa = halo.PrefixAttention(params_of(w), w.forest_csr(), "cuda")
    assert pa.plan.workspace_bytes > 0
    want, want_lse = pa.run(w.q, w.k_pool, w.v_pool)
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in range(2)]
    outs = [pa.alloc_outputs(w.q) for _ in streams]
    for _ in range(20):
        for s, (o, lse) in zip(streams, outs):
            pa.run(w.q, w.k_pool, w.v_pool, o, lse, stream=s)
    torch.cuda.synchronize()
    o, lse = pa.alloc_outputs(w.q)
    side = torch.cuda.Stream()
    call = pa.bind(w.q, w.k_pool, w.v_pool, o, lse, side)
    call()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        call()
    for _ in range(3):
        o.zero_()
        graph.replay()
        pa.run(w.q, w.k_pool, w.v_pool)   # eager work between the replays
        torch.cuda.synchronize()
        assert torch.equal(o, want) and torch.equal(lse, want_lse)
    for o, lse in outs:
        assert torch.equal(o, want) and torch.equal(lse, want_lse)


@pytest.mark.parametrize("dtype,n_new", [(torch.bfloat16, 40), (torch.bfloat16, 3), (torch.float32, 40),
                                         (torch.float32, 3)])
@pytest.mark.parametrize("where", ["q", "k", "v"])
def test_nan_inputs_stay_visible_through_the_pieces(gpu_lib, dtype, n_new, where):
    """A NaN in a query, a cached key or a cached value reaches exactly the
    outputs it belongs to, and LSE is -inf where the scores are NaN, in pieces
    (merged by rows and by workgroups) as uncut."""
    print(f"case: NaN in {where}, prefill {dtype} {n_new} tokens", flush=True)
    w = to_device(build_workload("nan", 74, 4, 2, 128, dtype, [6000, n_new], [[0, 1]], [n_new], value_scale=0.5))
    page = int(w.seg_pages[0][200])
    hit = np.zeros((n_new, 4, 128), bool)
    if where == "q":
        w.q[n_new - 1, 0, 5] = float("nan")
        hit[n_new - 1, 0] = True
    elif where == "k":
        w.k_pool[page, 0, 2, 7, 3] = float("nan")
        hit[:, :2] = True
    else:
        w.v_pool[page, 0, 9, 4] = float("nan")
        hit[:, :2, 9] = True
    pa = halo.PrefixAttention(params_of(w), w.forest_csr(), "cuda")
    assert pa.plan.workspace_bytes > 0
    o, lse = pa.run(w.q, w.k_pool, w.v_pool)
    o2, lse2 = pa.alloc_outputs(w.q)
    halo.prefix_attn_prefill(pa.plan, pa.meta, w.q, w.k_pool, w.v_pool, o2, lse2, None)
    for got, got_lse in ((o, lse), (o2, lse2)):
        assert (torch.isnan(got).cpu().numpy() == hit).all()
        assert (torch.isneginf(got_lse).cpu().numpy() == (hit.all(axis=2) if where != "v" else False)).all()
