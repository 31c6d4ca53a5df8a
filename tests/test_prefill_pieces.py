"""CPU checks of prefill plans whose items are cut into pieces (halo_plan.cpp):
for every output row the pieces' key ranges tile exactly the keys the row must
see, and every piece's rows have partial slots of their own."""

import numpy as np
import pytest
import torch

from paper_2509_02121_amd import halo
from test_abi_cpu import _expected_intervals, _params
from workloads import build_workload

PIECE = 2   # Item::flags of a piece


def _coverage(m, w):
    """(row, segment, end) of each maximal run of keys from 0, as the items of
    the plan cover them; fails on a gap, an overlap or a shared slot."""
    items = np.concatenate([m["items"].reshape(-1, 16), m["wide_items"].reshape(-1, 16)])
    items = items[items[:, 1] > 0]
    ranges, slots = {}, []
    for it in items:
        row0, n_rows, sp0, n_sp, kv_head, base, flags = it[0], it[1], it[2], it[3], it[4], it[5], it[7]
        assert (base >= 0) == bool(flags & PIECE)
        if base >= 0:
            slots.extend(range(base, base + n_rows))
        for r in m["rows"][row0:row0 + n_rows]:
            assert r[0] % w.num_q_heads // (w.num_q_heads // w.num_kv_heads) == kv_head
            for sp in m["spans"][sp0:sp0 + n_sp]:
                lo, hi = int(sp[1]), int(min(sp[2], r[1] + 1) if sp[3] else sp[2])
                if hi > lo:
                    ranges.setdefault((int(r[0]), int(sp[0])), []).append((lo, hi))
    assert len(slots) == len(set(slots)) and (not slots or max(slots) == len(slots) - 1)
    out = []
    for (row, seg), rs in ranges.items():
        rs.sort()
        assert rs[0][0] == 0 and all(a[1] == b[0] for a, b in zip(rs, rs[1:])), "gap or overlap"
        out.append((row, seg, rs[-1][1]))
    return sorted(out), len(slots)


@pytest.mark.parametrize("seed", range(12))
def test_pieces_tile_the_visible_keys(seed):
    rng = np.random.default_rng(seed)
    hkv, g = [(1, 4), (2, 1), (3, 2), (2, 8)][seed % 4]
    dtype = torch.bfloat16 if seed % 3 else torch.float32
    n = int(rng.integers(1, 4))
    shared = [int(x) for x in rng.integers(0, 1500, size=2)]
    own = [int(x) for x in rng.integers(0, 2500, size=n)]
    q_len = [int(x) for x in rng.integers(1, 300, size=n)]
    seg_len = shared + own + q_len
    paths = [[0, 1, 2 + r, 2 + n + r] if r else [2, 2 + n] for r in range(n)]
    w = build_workload("pieces", seed, hkv * g, hkv, 64, dtype, seg_len, paths, q_len)
    plan = halo.Plan.from_csr(_params(w), w.forest_csr())
    got, n_slots = _coverage(plan.inspect(), w)
    rows, segs, his = _expected_intervals(w)
    assert got == sorted(zip(rows.tolist(), segs.tolist(), his.tolist()))
    st = plan.stats()
    assert st["num_partial_rows"] == n_slots and (st["num_merge_rows"] > 0) == (n_slots > 0)
    pad = lambda x: -(-x // 256) * 256
    assert plan.workspace_bytes == (pad(n_slots * 64 * 4) + pad(n_slots * 4) if n_slots else 0)


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_kv_heads_share_their_spans(dtype):
    """The spans of a row block are listed once for all kv heads, cut into
    pieces or not: they are most of what the planner writes."""
    for q_len in ([64], [900, 3], [1] * 40):
        seg_len = [1500] + q_len
        paths = [[0, 1 + r] for r in range(len(q_len))]
        n = {}
        for h in (1, 8):
            params = halo.make_params(4 * h, h, 128, dtype, 1 << 16, 0.1)
            pages = [(x + 15) // 16 for x in seg_len]
            indptr = np.concatenate([[0], np.cumsum(pages)]).astype(np.int32)
            plan = halo.Plan(params, seg_len, indptr, np.arange(indptr[-1]), np.arange(len(q_len) + 1) * 2,
                             np.concatenate(paths), q_len)
            m = plan.inspect()
            items = np.concatenate([m["items"].reshape(-1, 16), m["wide_items"].reshape(-1, 16)])
            items = items[items[:, 1] > 0]
            assert len(m["spans"]) <= items[items[:, 4] == 0][:, 3].sum() * 2   # (with the uncut items')
            n[h] = len({(int(x[2]), int(x[3])) for x in items}), (items[:, 4] == 0).sum()
        assert n[1][0] == n[1][1] and n[8][0] == n[8][1]
