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


class _Spy:
    """The library, noting the workspace address of each prefill call."""

    def __init__(self, lib):
        self.lib, self.seen = lib, []

    def __getattr__(self, name):
        return getattr(self.lib, name)

    def halo_prefix_attn_prefill(self, *args):
        self.seen.append(args[7])
        return self.lib.halo_prefix_attn_prefill(*args)


def test_piecewise_prefill_on_two_streams_and_in_a_graph(gpu_lib, monkeypatch):
    """Calls of one object, each with its own queries: those that overlap on
    two streams have a workspace each, and so has every captured call, bound
    before its capture to one stream and replayed on another beside eager
    calls on the first."""
    print("case: prefill pieces on two streams, captured", flush=True)
    w = to_device(build_workload("streams", 73, 8, 2, 128, torch.bfloat16, [5000, 150], [[0, 1]], [150],
                                 value_scale=0.5))
    spy = _Spy(halo._LIB)
    monkeypatch.setattr(halo, "_LIB", spy)
    pa = halo.PrefixAttention(params_of(w), w.forest_csr(), "cuda")
    assert pa.plan.workspace_bytes > 0
    qs = [w.q * x for x in (1.0, -2.0, 0.5, 3.0, -1.0)]
    want = [pa.run(q, w.k_pool, w.v_pool) for q in qs]
    outs = [pa.alloc_outputs(q) for q in qs]
    side, other = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    spy.seen.clear()
    for _ in range(20):
        for i, s in ((0, side), (1, other)):
            pa.run(qs[i], w.k_pool, w.v_pool, *outs[i], stream=s)
    torch.cuda.synchronize()
    eager = set(spy.seen)
    assert len(eager) == 2
    # three callables of one stream, the first two captured
    calls = [pa.bind(qs[i], w.k_pool, w.v_pool, *outs[i], side) for i in (2, 3, 4)]
    calls[0]()
    torch.cuda.synchronize()
    graphs = []
    for call in calls[:2]:
        spy.seen.clear()
        graphs.append(torch.cuda.CUDAGraph())
        with torch.cuda.graph(graphs[-1], stream=side):
            call()
        assert len(spy.seen) == 1 and spy.seen[0] not in eager
        eager.add(spy.seen[0])
    bound = calls[2]
    del calls, call   # a graph needs nothing of its callable
    for _ in range(3):
        for o, lse in outs:
            o.zero_()
        torch.cuda.synchronize()
        with torch.cuda.stream(other):
            graphs[0].replay()
        graphs[1].replay()
        bound()
        for i, s in ((0, side), (1, other)):
            pa.run(qs[i], w.k_pool, w.v_pool, *outs[i], stream=s)
        torch.cuda.synchronize()
        for (o, lse), (wo, wl) in zip(outs, want):
            assert torch.equal(o, wo) and torch.equal(lse, wl)


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
