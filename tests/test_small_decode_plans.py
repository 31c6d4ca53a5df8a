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


@pytest.mark.parametrize("dtype,out_dtype", [(torch.float32, torch.float32), (torch.bfloat16, torch.float32)])
def test_a_cut_that_saves_less_than_the_merge_costs(dtype, out_dtype):
    """Rows of one short item each are not cut only to be merged; with a row
    that is merged anyway the chunks are short."""
    paths = [[i] for i in range(12)]
    assert _plan([75] * 12, paths, dtype, out_dtype).workspace_bytes == 0
    assert _plan([250] * 12, paths, dtype, out_dtype).workspace_bytes > 0
    m = _plan([75] * 11 + [300], paths, dtype, out_dtype).inspect()
    assert max(int(sp[2] - sp[1]) for sp in m["spans"]) <= 64


def test_rows_that_stay_whole_bound_the_cut():
    """Where a whole row's chain is as long as any other's, the others are not
    cut either (bf16 output); a shorter one does not stop the cut."""
    longest = lambda lens: max(int(sp[2] - sp[1]) for sp in _plan(
        lens, [[i] for i in range(len(lens))], torch.bfloat16, torch.bfloat16).inspect()["spans"])
    assert longest([250, 900, 900]) == 256
    assert longest([100, 900, 900]) == 100


def _covers(plan, csr):
    """Each request's items cover the keys of its path, each once."""
    m = plan.inspect()
    items = m["items"].reshape(-1, 16)
    got = {}
    for it, rec in zip(items, m["item_recs"].reshape(-1, 64)):
        if it[1] == 0:
            continue
        for k in range(it[3]):
            seg, kb, ke, _, off = (int(x) for x in m["spans"][it[2] + k][:5])
            assert kb <= ke
            if k == 0:
                assert (int(it[8]), int(it[9])) == (kb, ke)
                n = min(32, (ke - kb + 15) // 16)
                assert np.array_equal(rec[32:32 + n], m["page_ids"][off:off + n])
            for row in m["rows"][it[0]:it[0] + it[1], 0]:
                got.setdefault((int(row), seg), set()).update(range(kb, ke))
    paths = [csr["req_seg_ids"][a:b] for a, b in zip(csr["req_seg_indptr"][:-1], csr["req_seg_indptr"][1:])]
    for r, path in enumerate(paths):
        for s in path:
            for h in range(8):
                assert got.get((r * 8 + h, int(s)), set()) == set(range(int(csr["seg_len"][s])))
    for s, n in enumerate(csr["seg_len"]):
        ids = csr["seg_page_ids"][csr["seg_page_indptr"][s]:csr["seg_page_indptr"][s + 1]]
        off = m["seg_page_off"][s]
        assert np.array_equal(m["page_ids"][off:off + len(ids)], ids)


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("n", [250, 257, 440, 700])
def test_lengths_that_short_chunks_accept(n, dtype):
    """Removing tokens: a private segment of n keys takes every length above
    its last run of 256 keys, as with chunks of 256 keys, and grows again, on
    other pages too; one key less asks for a new plan."""
    paths = [[0, 1], [0, 2]]

    def forest(length, own):
        csr = _csr([700, length, 40], paths)
        csr["seg_page_ids"] = np.concatenate([np.arange(44), own, np.arange(500, 503)]).astype(np.int32)
        return csr

    own = np.arange(44, 44 + (n + 15) // 16)
    plan = halo.Plan.from_csr(halo.make_params(8, 2, 128, dtype, 1 << 16, 0.1), forest(n, own))
    low = (n - 1) // 256 * 256
    rng = np.random.default_rng(n)
    for step, length in enumerate([n - 1, low + 1, n, low + 33, n + 200, low + 2, low + 70, low + 16, n]):
        if length <= low:
            continue
        pages = (length + 15) // 16
        own = np.concatenate([own[:pages], 1000 + 100 * step + rng.permutation(100)[:max(0, pages - len(own))]])
        assert plan.update_lengths(forest(length, own)), (length, n)
        _covers(plan, forest(length, own))
    if low:
        assert not plan.update_lengths(forest(low, own[:low // 16]))
