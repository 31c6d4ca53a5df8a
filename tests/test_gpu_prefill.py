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
