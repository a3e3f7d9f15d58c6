"""The merge of a row block's splits by the workgroup that finishes last: few rows (the
splits spread over sets of threads, one batch and several) and many (chunks in batches of
four), at the edges between the two, for both element sizes and head sizes.  Repeated
launches find the arrival counters at zero again.  An infinite value of the last split stays
infinite."""
import numpy as np
import pytest
import torch

import synth
from gpu_common import run_fused
from test_gpu_parity import _both_paths

pytestmark = pytest.mark.gpu


# query rows of a row block: (query heads per kv-head) x suffix tokens
@pytest.mark.parametrize("heads,suffix_len,rows_per_block,head_dim,dtype,kv_splits", [
    (1, 1, 64, 128, "bf16", 2),       # 1 row: 16 chunks, two splits
    (4, 1, 64, 128, "bf16", 33),      # 4 rows, splits past one batch of each lane
    (4, 1, 64, 64, "f32", 9),
    (4, 2, 64, 128, "bf16", 17),      # 8 rows: 128 chunks, the most that spread over lanes
    (3, 3, 64, 128, "bf16", 5),       # 9 rows: 144 chunks, one a thread
    (4, 4, 64, 128, "bf16", 9),       # 16 rows: 256 chunks, a thread each, two batches
    (1, 17, 64, 128, "bf16", 9),      # 17 rows: 272 chunks, batches of four chunks
    (1, 17, 128, 64, "bf16", 5),      # 17 rows of 8 chunks, 512 threads
    (4, 25, 128, 128, "i8", 4),
    (4, 64, 256, 128, "bf16", 5),     # 256 rows, a second batch of one split
    (4, 61, 256, 64, "f32", 3),
])
def test_merge_in_kernel(heads, suffix_len, rows_per_block, head_dim, dtype, kv_splits):
    w = synth.small(pool_dtype=dtype, n_q_heads=2 * heads, n_kv_heads=2, head_dim=head_dim,
                    batch=2, chunks_per_req=4, chunk_len=700, keep=("ratio", 0.8, 0.9),
                    suffix_len=suffix_len, seed=71)
    opts = dict(rows_per_block=rows_per_block, kv_splits=kv_splits, merge_mode=1)
    plan = _both_paths(w, f"in-kernel merge {heads}x{suffix_len} {dtype} {opts}", **opts)
    assert plan.info["max_splits"] == kv_splits
    first, lse, _, dev = run_fused(w, plan=plan)
    for _ in range(3):
        out, l2, _, _ = run_fused(w, dev=dev, plan=plan)
        assert torch.equal(out, first) and torch.equal(l2, lse)


@pytest.mark.parametrize("heads,suffix_len,rows_per_block,dtype,kv_splits", [
    (4, 2, 64, "bf16", 3),            # splits spread over sets of threads
    (4, 2, 64, "f32", 2),
    (4, 25, 128, "bf16", 2),          # batches of four chunks and four splits
    (4, 61, 256, "bf16", 5),
    (3, 20, 64, "f32", 3),
])
def test_infinite_value_stays_infinite(heads, suffix_len, rows_per_block, dtype, kv_splits):
    """A value of +Inf at the first new token (which every row sees, in the last split)
    makes that channel +Inf in every row, and no other channel: no load that only fills a
    batch may meet it with weight 0."""
    w = synth.small(pool_dtype=dtype, n_q_heads=2 * heads, n_kv_heads=2, batch=2,
                    chunks_per_req=4, chunk_len=700, keep=("ratio", 0.8, 0.9),
                    suffix_len=suffix_len, seed=72)
    v = (w.v_suf if dtype == "f32" else synth.bf16_bits_to_f32(w.v_suf)).copy()
    v[:, 0, :, 5] = np.inf
    w = synth.with_overrides(w, v_suf=synth.cast_f64(v, w.act_dtype))
    for mode in (2, 1):
        out, _, plan, _ = run_fused(w, rows_per_block=rows_per_block, kv_splits=kv_splits,
                                    merge_mode=mode)
        assert plan.info["max_splits"] == kv_splits
        out = out.float()
        inf = torch.zeros_like(out, dtype=torch.bool)
        inf[..., 5] = True
        assert torch.equal(torch.isposinf(out), inf), mode
        assert torch.isfinite(out[~inf]).all(), mode
