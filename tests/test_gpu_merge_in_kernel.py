"""The merge of a row block's splits by the workgroup that finishes last: few rows (the
splits spread over sets of threads, one batch and several) and many (chunks in batches of
four), at the edges between the two, for both element sizes and head sizes.  Repeated
launches find the arrival counters at zero again."""
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
    (3, 3, 64, 128, "bf16", 5),       # 9 rows: 144 chunks, batches of four chunks
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
