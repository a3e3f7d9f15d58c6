"""Row blocks cut where a workgroup slot is full: splits of unequal length.

CPU: tests/work_split.cpp checks that the work lists of random ragged batches cover
every key tile of every row block exactly once, and that no row block that equal splits
would leave whole gets 16-bit partials.  GPU: few compute units are declared, so that small
batches are cut this way, for row blocks of each size and each key source."""
import os
import shutil
import subprocess

import numpy as np
import pytest
import torch  # noqa: F401  (before the library, so that both share one HIP runtime)

import paper_2607_17715_amd as c2kv
import synth

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ is not installed")
def test_work_list_covers_every_tile_once(tmp_path):
    exe = str(tmp_path / "work_split")
    csrc = os.path.join(ROOT, "paper_2607_17715_amd", "csrc")
    subprocess.run(["g++", "-std=c++17", "-O2", "-I", os.path.join(ROOT, "include"), "-I", csrc,
                    os.path.join(ROOT, "tests", "work_split.cpp"),
                    os.path.join(csrc, "plan.cpp"), "-o", exe], check=True, timeout=300)
    r = subprocess.run([exe, "400", "3"], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout[-2000:]
    # counts that equal splits alone would leave at 0
    words = r.stdout.split()
    assert int(words[3]) > 60 and int(words[5]) > 5, r.stdout


CASES = [
    # 64-row blocks, paged and pool: one row block per (request, kv-head)
    (dict(batch=5, n_q_heads=8, n_kv_heads=4, suffix_len=2, chunks_per_req=4, chunk_len=400), 8),
    # 128-row blocks, int8
    (dict(batch=5, n_q_heads=8, n_kv_heads=2, suffix_len=29, chunks_per_req=4, chunk_len=400,
          pool_dtype="i8"), 8),
    # 256-row blocks, the last of a request short, head_dim 64
    (dict(batch=5, n_q_heads=12, n_kv_heads=4, suffix_len=101, chunks_per_req=4, chunk_len=500,
          head_dim=64), 32),
    # fp32
    (dict(batch=3, n_q_heads=4, n_kv_heads=4, suffix_len=70, chunks_per_req=4, chunk_len=500,
          pool_dtype="f32"), 8),
]


def test_one_round_of_even_splits_is_kept():
    """24 fp32 row blocks of 256 rows, 5 to 17 tiles each: pieces of one and two tiles fit one
    round of 256 slots, so they are not cut into fewer and longer ones."""
    w = synth.small(pool_dtype="f32", n_q_heads=8, n_kv_heads=2, batch=1, chunks_per_req=2,
                    keep=("count", 130), prefix_len=0, suffix_len=744, seed=3)
    i = c2kv.Plan.for_workload(w).info
    assert i["rows_per_block"] == 256 and i["n_merge_groups"] == 24
    assert 200 < i["n_work_items"] <= 256, i


def test_decode_partials_hold_the_rows_that_exist():
    """560 decode row blocks of 4 rows on 512 slots, whole by equal splits, are cut: their
    fp32 pieces take 16 of a row block's 64 rows, and so fit the static scratch."""
    n, b = 3700, 70
    plan = c2kv.Plan(32, 8, 128, "bf16", 5e5, np.arange(b + 1, dtype=np.int32),
                     np.zeros(b, np.int64), np.full(b, n, np.int32), np.zeros(b, np.int32),
                     n * np.arange(b + 1, dtype=np.int32), np.tile(np.arange(n, dtype=np.int32), b),
                     1)
    i = plan.info
    assert i["rows_per_block"] == 64 and i["n_merge_groups"] > 0 and i["n_work_items"] > 560, i
    assert i["workspace_bytes"] <= c2kv.STATIC_SCRATCH_BYTES


@pytest.mark.gpu
@pytest.mark.parametrize("shape,num_cus", CASES)
def test_cut_row_blocks_parity(shape, num_cus):
    from test_gpu_parity import _both_paths
    w = synth.small(seed=31, keep=("ratio", 0.4, 0.9), **shape)
    plan = _both_paths(w, f"cut {shape}", num_cus=num_cus)
    i = plan.info
    groups = w.batch * w.n_kv_heads * -(-w.suffix_len * (w.n_q_heads // w.n_kv_heads) //
                                        i["rows_per_block"])
    # equal splits would leave all of them whole: there is a row block per slot
    assert groups >= num_cus * (2 if i["rows_per_block"] == 64 else 1)
    assert i["n_merge_groups"] > 0 and i["n_work_items"] > groups, (groups, i)


@pytest.mark.gpu
@pytest.mark.parametrize("shape,num_cus", CASES[:3])
def test_cut_row_blocks_round_once(shape, num_cus):
    """Row blocks that equal splits would leave whole (at least one per slot) are rounded
    to bf16 once, as they are when whole.  With q = 0 every probability is exactly 1, so
    that an output is the mean of values drawn from [1, 2) and nothing but its own
    rounding, half a unit of 2^-7, and fp32 sums (relative 2^-24 for each of about 100
    steps, and the weights' 1e-6: 1e-5 of values below 2) separate it from float64."""
    from gpu_common import oracle_ref, run_fused, run_paged
    w = synth.small(seed=33, keep=("ratio", 0.4, 0.9), **dict(shape, pool_dtype="bf16"))
    rng = np.random.default_rng(7)
    values = lambda a: synth.cast_f64(1 + rng.integers(0, 128, a.shape) / 128, "bf16")
    w = synth.with_overrides(w, q=np.zeros_like(w.q), pool_v=values(w.pool_v),
                             v_suf=values(w.v_suf))
    ref, _, _ = oracle_ref(w)
    out, _, plan, dev = run_fused(w, num_cus=num_cus)
    assert plan.info["n_merge_groups"] > 0
    paged, _, _, _, _ = run_paged(w, dev=dev, plan=plan)
    assert torch.equal(out, paged)
    assert np.abs(c2kv.to_numpy_f64(out) - ref).max() <= 2.0 ** -8 + 2e-5


@pytest.mark.gpu
@pytest.mark.parametrize("shape,opts", [
    # fp32 pieces of 64- and 256-row blocks, combined by the merge kernel
    (CASES[0][0], dict(num_cus=8, merge_mode=2)),
    (CASES[2][0], dict(num_cus=32, merge_mode=2)),
    # more than 16 pieces of few rows: one row a workgroup
    (dict(n_q_heads=4, n_kv_heads=1, batch=3, chunks_per_req=4, chunk_len=3500, suffix_len=3,
          seed=0), dict(num_cus=37)),
    # 96 row blocks in 256 pieces, which fit the static scratch only with some in bf16
    (dict(n_q_heads=8, n_kv_heads=8, batch=4, chunks_per_req=1, chunk_len=310, prefix_len=0,
          keep=("ratio", 0.9, 1.0), suffix_len=744, seed=5), dict(merge_mode=1)),
    (dict(n_q_heads=8, n_kv_heads=8, batch=4, chunks_per_req=1, chunk_len=310, prefix_len=0,
          keep=("ratio", 0.9, 1.0), suffix_len=744, seed=5), dict(merge_mode=2)),
])
def test_fp32_pieces_parity(shape, opts):
    from gpu_common import run_fused
    from test_gpu_parity import _both_paths
    w = synth.small(**dict(dict(seed=31, keep=("ratio", 0.4, 0.95)), **shape))
    plan = _both_paths(w, f"fp32 pieces {shape}", **opts)
    i = plan.info
    rows = min(i["rows_per_block"], -(-w.suffix_len * w.n_q_heads // w.n_kv_heads // 16) * 16)
    bf16 = i["n_work_items"] * rows * w.head_dim * 2
    assert i["n_merge_groups"] > 0 and bf16 < i["workspace_bytes"] <= c2kv.STATIC_SCRATCH_BYTES
    assert (i["max_splits"] > 16) == (shape.get("chunk_len") == 3500)
    # the same bits from the static scratch, and from replays of a graph
    ref, ref_lse, _, dev = run_fused(w, plan=plan)
    out, lse = dev.out_like(), dev.lse_like()
    c2kv.c2kv_compose_attend_static(plan, dev.pool, dev.q, dev.k_suf, dev.v_suf, out, lse)
    torch.cuda.synchronize()
    assert torch.equal(out, ref) and torch.equal(lse, ref_lse)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        c2kv.c2kv_compose_attend(plan, dev.pool, dev.q, dev.k_suf, dev.v_suf, out, lse)
    for _ in range(3):
        out.zero_()
        lse.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, ref) and torch.equal(lse, ref_lse)
        run_fused(w, dev=dev, plan=plan)
