"""Value tiles read by whole rows and transposed as words of two keys: key counts at the
edges of a pair and of a 64-key tile, for each storage, head size and row-block size.  The
composed pages are compared with the oracle's, the tail of the last tile with zero."""
import numpy as np
import pytest

import paper_2607_17715_amd as c2kv
import synth
from gpu_common import Dev, compare, oracle_ref, run_fused, run_paged, say
from test_gpu_parity import _check_pages

pytestmark = pytest.mark.gpu

KEY_TILE = 64


@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("pool_dtype", ["bf16", "i8", "f32"])
@pytest.mark.parametrize("kept,suffix_len", [(1, 1), (2, 64), (63, 65), (64, 3), (65, 63),
                                             (129, 127)])
def test_value_rows(head_dim, pool_dtype, kept, suffix_len):
    w = synth.small(pool_dtype=pool_dtype, head_dim=head_dim, n_q_heads=6, n_kv_heads=2, batch=2,
                    prefix_len=0, chunks_per_req=1, keep=("count", kept), suffix_len=suffix_len,
                    seed=17)
    what = f"value rows {pool_dtype} D={head_dim} N={kept} S={suffix_len}"
    ref_out, ref_lse, _ = oracle_ref(w)
    dev = Dev(w)
    for rows in (64, 128, 256):
        say(f"{what} rows_per_block={rows}")
        out, lse, plan, _ = run_fused(w, dev=dev, rows_per_block=rows)
        compare(w, out, lse, ref_out, ref_lse, what=what)
    _, _, plan, _, res = run_paged(w, dev=dev, page_size=128)
    _check_pages(w, plan, res)
    end = -(-kept // KEY_TILE) * KEY_TILE
    bt, ps = plan.block_table(), plan.info["page_size"]
    s = np.arange(kept, end)
    vp = c2kv.to_numpy_f64(res["v_pages"])
    for b in range(w.batch):
        assert (vp[bt[b][s // ps], :, :, s % ps] == 0).all(), (what, b)
