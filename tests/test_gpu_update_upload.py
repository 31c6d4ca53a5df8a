"""GPU checks of the metadata uploads between decode steps: after any sequence
of in-place updates (growing and shrinking, pages opened and dropped) each
double buffer holds what a whole upload of the plan would."""

import numpy as np
import pytest
import torch

from gpu_helpers import assert_parity, oracle_for, params_of, to_device
from paper_2509_02121_amd import halo
from workloads import build_workload

pytestmark = pytest.mark.gpu


def _shortened(csr, w, cut):
    """The forest with `cut` tokens fewer per segment, pages dropped with them."""
    out = {k: (v.copy() if v is not None else None) for k, v in csr.items()}
    out["seg_len"] = (csr["seg_len"] - cut).astype(np.int32)
    pages = [w.seg_pages[s][:(int(n) + 15) // 16] for s, n in enumerate(out["seg_len"])]
    out["seg_page_indptr"] = np.concatenate([[0], np.cumsum([len(p) for p in pages])]).astype(np.int32)
    out["seg_page_ids"] = np.concatenate(pages).astype(np.int32)
    return out


@pytest.mark.parametrize("where", ["current stream", "copy stream", "own stream"])
@pytest.mark.parametrize("dtype,n_req,private", [(torch.bfloat16, 9, 300), (torch.bfloat16, 3, 1500),
                                                 (torch.float32, 5, 120)])
def test_updates_reach_both_buffers(gpu_lib, where, dtype, n_req, private):
    print(f"case: update uploads {where} {dtype} {n_req} x {private}", flush=True)
    rng = np.random.default_rng(n_req)
    seg_len = [200] + [int(x) for x in rng.integers(private, private * 5 // 4, size=n_req)]
    w = to_device(build_workload("updates", 91, 8, 2, 64, dtype, seg_len, [[0, 1 + r] for r in range(n_req)],
                                 value_scale=0.5))
    full = w.forest_csr()
    pa = halo.PrefixAttention(params_of(w), _shortened(full, w, np.array([0] + [60] * n_req)), "cuda")
    pa.IN_ORDER_KV_BYTES = 0 if where == "copy stream" else pa.IN_ORDER_KV_BYTES
    stream = torch.cuda.Stream() if where == "own stream" else None
    whole = torch.empty_like(pa.meta)
    applied = 0
    for low, high in ((40, 60), (20, 41), (0, 3), (0, 1), (30, 31), (10, 55), (0, 20), (0, 1)):
        cut = np.array([0] + [int(x) for x in rng.integers(low, high, size=n_req)])
        applied += pa.update(_shortened(full, w, cut), stream)
        o, lse = pa.run(w.q, w.k_pool, w.v_pool)
        if whole.numel() < pa.plan.device_meta_bytes:
            whole = torch.empty_like(pa.meta)
        pa.plan.upload(whole)
        o2, lse2 = pa.alloc_outputs(w.q)
        halo.prefix_attn_decode(pa.plan, whole, w.q, w.k_pool, w.v_pool, o2, lse2, pa.workspace)
        torch.cuda.synchronize()
        assert torch.equal(o, o2) and torch.equal(lse, lse2), f"cut {cut}"
        assert not torch.isnan(o).any()
    assert applied >= 6, "updates are mostly in place"


def test_captured_upload_follows_the_plan(gpu_lib):
    """A captured update upload copies, on each replay, the image as the plan
    has it by then."""
    print("case: captured update upload", flush=True)
    seg_len = [200, 330, 310, 350]
    w = to_device(build_workload("updates", 92, 8, 2, 64, torch.bfloat16, seg_len, [[0, 1], [0, 2], [0, 3]],
                                 value_scale=0.5))
    full = w.forest_csr()
    pa = halo.PrefixAttention(params_of(w), _shortened(full, w, np.array([0, 60, 60, 60])), "cuda")
    plan, meta = pa.plan, pa.meta
    assert plan.update_lengths(_shortened(full, w, np.array([0, 50, 52, 50])))
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=side):
        plan.upload_update(meta, side)
    whole = torch.empty_like(meta)
    for cut in (50, 31, 12, 33, 0):
        assert plan.update_lengths(_shortened(full, w, np.array([0, cut, cut // 2, cut])))
        g.replay()
        plan.upload(whole)
        torch.cuda.synchronize()
        (o, lse), (o2, lse2) = pa.alloc_outputs(w.q), pa.alloc_outputs(w.q)
        halo.prefix_attn_decode(plan, meta, w.q, w.k_pool, w.v_pool, o, lse, pa.workspace)
        halo.prefix_attn_decode(plan, whole, w.q, w.k_pool, w.v_pool, o2, lse2, pa.workspace)
        torch.cuda.synchronize()
        assert torch.equal(o, o2) and torch.equal(lse, lse2), f"cut {cut}"


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_removed_tokens_reach_both_buffers(gpu_lib, dtype):
    """Tokens are removed past the starts of short key chunks (whose spans are
    then empty) and appended again: each update applies
    and its upload gives the bits of a whole upload and the oracle's values."""
    print(f"case: removed tokens {dtype}", flush=True)
    seg_len = [200, 250, 510, 300]
    w = to_device(build_workload("removed", 93, 8, 2, 128, dtype, seg_len, [[0, 1], [0, 2], [0, 3]],
                                 value_scale=0.5 if dtype == torch.bfloat16 else 1.0))
    full = w.forest_csr()
    pa = halo.PrefixAttention(params_of(w), full, "cuda")
    whole = torch.empty_like(pa.meta)
    cuts = [[1, 1, 1], [249, 253, 43], [60, 100, 3], [0, 0, 0], [200, 190, 20], [130, 64, 40], [0, 0, 0]]
    for cut in cuts:
        csr = _shortened(full, w, np.array([0] + cut))
        assert pa.update(csr), cut
        o, lse = pa.run(w.q, w.k_pool, w.v_pool)
        pa.plan.upload(whole)
        o2, lse2 = pa.alloc_outputs(w.q)
        halo.prefix_attn_decode(pa.plan, whole, w.q, w.k_pool, w.v_pool, o2, lse2, pa.workspace)
        torch.cuda.synchronize()
        assert torch.equal(o, o2) and torch.equal(lse, lse2), f"cut {cut}"
        saved = w.seg_len
        w.seg_len = csr["seg_len"]
        ro, rl, rows = oracle_for(w)
        w.seg_len = saved
        assert_parity(w, o.double().cpu().numpy(), lse.double().cpu().numpy(), ro, rl, rows, f"cut {cut}")


def _small(seed, n_req=3):
    seg_len = [200] + [330 + 7 * r for r in range(n_req)]
    return to_device(build_workload("updates", seed, 8, 2, 64, torch.bfloat16, seg_len,
                                    [[0, 1 + r] for r in range(n_req)], value_scale=0.5))


def test_uploads_go_in_order_only_on_the_stream_of_all_calls(gpu_lib):
    """An upload is put on the current stream only if every call of the object
    was there and the GPU is not behind: a decode on a second stream never
    waits for what the current one holds. (By the stream chosen; streams that
    share a hardware queue wait for each other whatever is chosen.)"""
    print("case: the stream of an upload", flush=True)
    w = _small(94)
    full = w.forest_csr()
    cut = [_shortened(full, w, np.array([0] + [c] * 3)) for c in (9, 8, 7, 6)]
    second = torch.cuda.Stream()

    def uploads(pa, streams):
        """The stream of each update's upload, runs on the streams given."""
        used = []
        for csr, s in zip(cut, streams):
            torch.cuda.synchronize()   # the GPU is not behind
            assert pa.update(csr)
            used.append(pa._upload_streams[pa._cur])
            pa.run(w.q, w.k_pool, w.v_pool, stream=s)
        torch.cuda.synchronize()
        return used

    now = torch.cuda.current_stream()
    pa = halo.PrefixAttention(params_of(w), full, "cuda")
    assert uploads(pa, [second] * 4) == [pa._copy_stream] * 4
    pa = halo.PrefixAttention(params_of(w), full, "cuda")
    # (no call yet: nothing says where they will be)
    assert uploads(pa, [None, None, second, None]) == [pa._copy_stream, now, now, pa._copy_stream]
    assert uploads(pa, [None] * 4) == [pa._copy_stream] * 4
    pa = halo.PrefixAttention(params_of(w), full, "cuda")
    pa.run(w.q, w.k_pool, w.v_pool)
    assert pa.update(cut[0], second) and pa._upload_streams[pa._cur] == second   # as given


def test_uploads_of_many_plans_at_once(gpu_lib):
    """More uploads in flight than there are staging buffers, on as many
    streams: each buffer holds what a whole upload gives."""
    print("case: uploads of many plans", flush=True)
    w = _small(95)
    full = w.forest_csr()
    short = _shortened(full, w, np.array([0, 60, 60, 60]))
    plans = [halo.Plan.from_csr(params_of(w), short) for _ in range(12)]
    metas = [torch.empty(p.device_meta_bytes, dtype=torch.uint8, device="cuda") for p in plans]
    streams = [torch.cuda.Stream() for _ in plans]
    for p, m in zip(plans, metas):
        p.upload(m)
    torch.cuda.synchronize()
    # pages that open again after a removal are others than before
    owned = [[list(x) for x in np.split(short["seg_page_ids"], short["seg_page_indptr"][1:-1])] for _ in plans]
    fresh = w.num_pool_pages - 1
    for cut in (50, 31, 55, 33, 0, 12, 60, 0):
        for i, (p, m, s) in enumerate(zip(plans, metas, streams)):
            csr = _shortened(full, w, np.array([0, cut, (cut + 7 * i) % 61, cut]))
            for seg, n in enumerate(csr["seg_len"]):
                pages = owned[i][seg][:(int(n) + 15) // 16]
                while len(pages) < (int(n) + 15) // 16:
                    pages.append(fresh)
                    fresh = fresh - 1 if fresh else w.num_pool_pages - 1
                owned[i][seg] = pages
            csr["seg_page_ids"] = np.concatenate(owned[i]).astype(np.int32)
            assert p.update_lengths(csr)
            p.upload_update(m, s)
    torch.cuda.synchronize()
    for p, m in zip(plans, metas):
        assert m.cpu().numpy().tobytes() == p.image()
