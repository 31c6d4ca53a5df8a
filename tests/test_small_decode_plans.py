"""Plans of small decode batches (CPU): the key chunks are shortened, but rows
that one item would hold at the default chunks are not cut where a cut would
round them to bf16 twice."""

import numpy as np
import pytest
import torch

from paper_2509_02121_amd import halo


def _csr(seg_len, paths):
    pages = [(n + 15) // 16 for n in seg_len]
    indptr = np.concatenate([[0], np.cumsum(pages)]).astype(np.int32)
    req = np.concatenate([[0], np.cumsum([len(p) for p in paths])]).astype(np.int32)
    return dict(seg_len=np.array(seg_len, np.int32), seg_page_indptr=indptr,
                seg_page_ids=np.arange(indptr[-1], dtype=np.int32), req_seg_indptr=req,
                req_seg_ids=np.concatenate([np.array(p, np.int32) for p in paths]), q_len=None)


def _plan(seg_len, paths, dtype, out_dtype, options=None):
    params = halo.make_params(8, 2, 128, dtype, 1 << 16, 0.1, out_dtype)
    return halo.Plan.from_csr(params, _csr(seg_len, paths), options)


@pytest.mark.parametrize("seg_len,paths", [
    ([200], [[0]]), ([256] * 16, [[i] for i in range(16)]), ([512], [[0]] * 4), ([500, 0, 0], [[0, 1], [0, 2]]),
    ([96, 60, 90, 256], [[0, 1, 2], [3]])])
def test_rows_of_one_item_are_rounded_once(seg_len, paths):
    plan = _plan(seg_len, paths, torch.bfloat16, torch.bfloat16)
    assert plan.stats()["num_partial_rows"] == 0 and plan.workspace_bytes == 0
    # an fp32 output loses nothing by a cut
    for dtype in (torch.bfloat16, torch.float32):
        assert _plan(seg_len, paths, dtype, torch.float32).stats()["num_partial_rows"] > 0
    # the caller's own chunk lengths apply to every row
    cut = _plan(seg_len, paths, torch.bfloat16, torch.bfloat16, {"kc_private": 32, "kc_shared": 32})
    assert cut.stats()["num_partial_rows"] > 0


def test_only_those_rows_stay_whole():
    """Beside requests of one item, the others' chunks are short: private keys
    of more than 256, a shared segment that has private keys beside it."""
    seg_len = [250, 257, 1000, 40, 50]
    paths = [[0], [1], [2, 3], [2, 4]]
    plan = _plan(seg_len, paths, torch.bfloat16, torch.bfloat16)
    m = plan.inspect()
    merged = {int(r) // 8 for r in m["merge_rows"]}
    assert merged == {1, 2, 3}
    longest = {}
    for sp in m["spans"]:
        longest[int(sp[0])] = max(longest.get(int(sp[0]), 0), int(sp[2] - sp[1]))
    assert longest[0] == 250 and longest[1] <= 64 and longest[2] <= 64
    # one request that has only the shared segment, of one default chunk, keeps
    # it whole for all
    m = _plan([400, 40, 50], [[0], [0, 1], [0, 2]], torch.bfloat16, torch.bfloat16).inspect()
    assert max(int(sp[2] - sp[1]) for sp in m["spans"] if sp[0] == 0) == 400
